// wait_for_word with a stubbed word, stream and clock: each way it can end.  Prints the number of checks; ends with an error at the first that fails.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "star_wait.h"

using namespace star;

namespace {
int checks = 0;
void check(bool ok, const char* what) {
    ++checks;
    if (ok) return;
    std::fprintf(stderr, "failed: %s\n", what);
    std::exit(1);
}

struct Stub {
    long looks = 0, pauses = 0, asks = 0;
    long written_at_look = -1, written_at_pause = -1, written_at_ask = -1;   // -1: never
    std::vector<Ask> answers;                                                // the last one for good
    bool done() const {
        return (written_at_look >= 0 && looks >= written_at_look) || (written_at_pause >= 0 && pauses >= written_at_pause) ||
               (written_at_ask >= 0 && asks >= written_at_ask);
    }
    WaitEnd run() {
        return wait_for_word([&] { ++looks; return done(); },
                             [&] { const Ask a = answers[(size_t)asks < answers.size() ? asks : answers.size() - 1]; ++asks; return a; },
                             [&] {
                                 ++pauses;
                                 if (pauses > 1000L * 1000 * 1000) std::exit(2);   // no end
                             });
    }
};
}  // namespace

int main() {
    Stub s;
    s.written_at_look = 1;
    s.answers = {Ask::Failed};
    check(s.run() == WaitEnd::Written && s.pauses == 0 && s.asks == 0, "a word that is there costs a look");

    s = Stub();
    s.written_at_pause = kPausesPerAsk / 2;
    s.answers = {Ask::Failed};
    check(s.run() == WaitEnd::Written && s.asks == 0, "a word soon after the spins costs no question");

    s = Stub();
    s.written_at_pause = 50L * kPausesPerAsk + 3;
    s.answers = {Ask::Busy};
    check(s.run() == WaitEnd::Written && s.asks == 50, "a busy stream is waited for");

    s = Stub();
    s.written_at_pause = 10L * 1000 * 1000;
    s.answers = {Ask::Busy};
    check(s.run() == WaitEnd::Written, "however long it is busy");

    s = Stub();
    s.answers = {Ask::Busy, Ask::Busy, Ask::Failed};
    check(s.run() == WaitEnd::Failed && s.asks == 3, "a failed stream ends the wait at once");

    s = Stub();
    s.written_at_ask = 1;
    s.answers = {Ask::Failed};
    check(s.run() == WaitEnd::Written, "not if the word has been written meanwhile");

    s = Stub();
    s.answers = {Ask::Idle};
    check(s.run() == WaitEnd::Untold && s.asks == kIdleAsks, "an idle stream writes no word any more");

    s = Stub();
    s.answers.assign(kIdleAsks - 1, Ask::Idle);
    s.answers.push_back(Ask::Busy);
    s.written_at_ask = 2L * kIdleAsks;
    check(s.run() == WaitEnd::Written, "a stream that goes on being busy does");

    s = Stub();
    s.answers = {Ask::Unknown};
    check(s.run() == WaitEnd::Failed && s.asks == kUnknownAsks, "a stream that may not be asked ends the wait late");

    s = Stub();
    s.answers = {Ask::Unknown};
    s.written_at_ask = kUnknownAsks - 1;
    check(s.run() == WaitEnd::Written, "and is waited for until then");

    std::printf("%d checks passed\n", checks);
    return 0;
}
