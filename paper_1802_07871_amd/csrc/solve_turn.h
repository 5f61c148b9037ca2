// solve_turn.h -- one-launch solves of a process that share a device (included
// by ctbop.hip).
//
// The blocks of a one-launch solve wait for each other, so they have to be on
// the device together.  Two solves on two streams that do not fit at once can
// each hold the CUs that the other's last blocks need, until a wait runs out
// (four threads, 12,000 atoms each: 66 ms per evaluation, 1.8 with the order
// below).  Here every solve states the CUs it may hold; one that does not fit
// beside those in flight has its stream wait for the oldest of them.  Nobody
// waits on the host, a lone caller makes no further API call, and small
// systems still run side by side.
#pragma once

namespace {

constexpr int TURN_DEVICES = 64;
// Consecutive blocks go to the device's XCDs in turn, so a solve is counted by
// its share of one: ceil(blocks / 8) of ncu / 8 CUs (no fewer blocks than a
// device of fewer XCDs would hold).
constexpr int TURN_XCDS = 8;

struct SolveTurn {
    struct Entry {
        const void *who;
        hipStream_t st;            // stream of the solve, recorded by whoever waits for it, or
        hipEvent_t done;           // an event recorded after the solve
        int share;
    };
    std::mutex mu;
    std::vector<Entry> on;
    hipEvent_t ev = nullptr;       // while users > 0
    int users = 0;
};
SolveTurn solve_turns[TURN_DEVICES];

// The device's event, for a context (with its side stream) or a server; dev is
// set to the device, and leave_turn takes it back.
int join_turn(int &dev)
{
    int d = -1;
    HIPCHK(hipGetDevice(&d));
    if (d < 0 || d >= TURN_DEVICES) return CTBOP_OK;
    SolveTurn &T = solve_turns[d];
    std::lock_guard<std::mutex> lk(T.mu);
    if (T.users == 0) HIPCHK(hipEventCreateWithFlags(&T.ev, hipEventDisableTiming));
    T.users++;
    dev = d;
    return CTBOP_OK;
}
void leave_turn(int &dev)
{
    if (dev < 0) return;
    SolveTurn &T = solve_turns[dev];
    std::lock_guard<std::mutex> lk(T.mu);
    if (--T.users == 0) {
        (void)hipEventDestroy(T.ev);
        T.ev = nullptr;
    }
    dev = -1;
}

// One call's solve: enter() before its launch, launched() after it, and
// leave() (or the end of the scope) once the host knows it has ended.
class SolvePass {
    SolveTurn *T = nullptr;
    std::unique_lock<std::mutex> lk;
    hipStream_t st = nullptr;
    int share = 0;
    bool listed = false;

public:
    int enter(int blocks, int ncu, hipStream_t stream)
    {
        int d = -1;
        HIPCHK(hipGetDevice(&d));
        if (d < 0 || d >= TURN_DEVICES) return CTBOP_OK;
        const int room = std::max(1, ncu / TURN_XCDS);
        st = stream;
        share = std::min((blocks + TURN_XCDS - 1) / TURN_XCDS, room);
        lk = std::unique_lock<std::mutex>(solve_turns[d].mu);
        T = &solve_turns[d];
        int used = share;
        for (const auto &e : T->on) used += e.share;
        for (const auto &e : T->on) {
            if (used <= room) break;
            used -= e.share;
            if (!e.done && e.st == st) continue;
            // (an event waited for may be recorded anew: a wait keeps the record it found)
            if (!e.done) {
                if (!T->ev) continue;
                HIPCHK(hipEventRecord(T->ev, e.st));
            }
            HIPCHK(hipStreamWaitEvent(st, e.done ? e.done : T->ev, 0));
        }
        return CTBOP_OK;
    }
    // done: an event to record after the solve, for a caller whose stream goes
    // on with other work
    int launched(hipEvent_t done = nullptr)
    {
        if (!T) return CTBOP_OK;
        if (done) HIPCHK(hipEventRecord(done, st));
        // (the handle of a thread's own stream means another stream to other
        // threads: these wait on the host instead)
        if (!done && st == hipStreamPerThread) return CTBOP_OK;
        T->on.push_back({this, st, done, share});
        listed = true;
        lk.unlock();
        return CTBOP_OK;
    }
    void leave()
    {
        if (!T) return;
        if (!lk.owns_lock()) lk.lock();
        if (listed)
            for (auto it = T->on.begin(); it != T->on.end(); ++it)
                if (it->who == this) {
                    T->on.erase(it);
                    break;
                }
        listed = false;
        lk.unlock();
        T = nullptr;
    }
    ~SolvePass() { leave(); }
};

} // namespace
