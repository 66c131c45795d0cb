// How the host waits for a word that a kernel writes, without HIP (built into a test of its own as well).
#pragma once
#include <cstdint>

namespace star {

// What a look at the stream behind the word says.
enum class Ask {
    Busy,     // there is work on it
    Idle,     // there is none
    Unknown,  // it cannot be asked (it is being captured, or its handle is no longer one)
    Failed    // the stream or its device reports an error
};

enum class WaitEnd {
    Written,
    Failed,   // Ask::Failed, or for too long Ask::Unknown
    Untold    // the stream has been idle for long, and the word is not written: nobody is left to write it
};

constexpr int kSpins = 20000;         // about 0.1 ms: eight calls ahead of a short shard's kernels
constexpr int kPausesPerAsk = 100;    // of 10 us and more each
// An idle stream's kernels have written the word.  The handle may be another stream's by now, though, if the caller has destroyed its own
// with work left on it: that work gets this many looks more (six seconds, one at the least).
constexpr int kIdleAsks = 1000;
constexpr int kUnknownAsks = 20000;   // (two minutes, 20 s at the least)

// Returns when written() holds, or when it cannot be expected to hold any more.  pause() sleeps.
template <class Written, class AskStream, class Pause>
WaitEnd wait_for_word(Written&& written, AskStream&& ask, Pause&& pause) {
    for (int i = 0; i < kSpins; ++i)
        if (written()) return WaitEnd::Written;
    for (int idle = 0, unknown = 0;;) {
        for (int i = 0; i < kPausesPerAsk; ++i) {
            pause();
            if (written()) return WaitEnd::Written;
        }
        const Ask a = ask();
        if (written()) return WaitEnd::Written;   // (between the last look and the question)
        idle = a == Ask::Idle ? idle + 1 : 0;
        unknown = a == Ask::Unknown ? unknown + 1 : 0;
        if (a == Ask::Failed || unknown >= kUnknownAsks) return WaitEnd::Failed;
        if (idle >= kIdleAsks) return WaitEnd::Untold;
    }
}

}  // namespace star
