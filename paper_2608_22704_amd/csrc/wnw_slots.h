// Scratch slots that launches of any stream and thread of a device share, host side: which slot a launch
// may use without waiting for another stream.  No GPU header here: the runtime's calls come through RT
// (Stream, Event, Error; ok, create, query, wait, record, shared_handle), so that the rule runs on the CPU too.
#pragma once

#include <mutex>

namespace wnw {

template <class RT, int N>
class SlotPool {
public:
    // Calls launch(slot), which enqueues the slot's next user on `st`, and returns true; `err` is the first
    // failure of the launch or of the event after it.  Returns false, with nothing enqueued, when every slot
    // may still be in use by another stream: the caller then does without one.
    template <class Launch>
    bool run(typename RT::Stream st, typename RT::Error &err, Launch launch)
    {
        std::lock_guard<std::mutex> lk(mu_);
        const int i = pick(st);
        if (i < 0) return false;
        err = launch(i);
        if (!RT::ok(err)) return true;   // nothing was enqueued: the slot is as it was
        err = RT::record(slot_[i].done, st);
        slot_[i].last = st;
        // without its event nobody can tell when the launch ends
        slot_[i].state = RT::ok(err) ? USED : LOST;
        return true;
    }

private:
    enum State { NEW, USED, LOST };
    struct Slot {
        typename RT::Event done{};       // recorded after the slot's last user
        typename RT::Stream last{};
        State state = NEW;
    };

    int pick(typename RT::Stream st)
    {
        // The slot that this stream used last: the stream itself orders the two launches, so the wait costs
        // nothing and depends on nobody else (it is there for a handle value that a new stream got from a
        // destroyed one).  A handle that several streams share does not tell them apart.
        if (!RT::shared_handle(st))
            for (int i = 0; i < N; ++i)
                if (slot_[i].state == USED && slot_[i].last == st) {
                    if (RT::ok(RT::wait(st, slot_[i].done))) return i;
                    slot_[i].state = LOST;   // the event is gone (a device reset)
                }
        // else one whose last user has ended, else a new one; never one to wait for
        for (int i = 0; i < N; ++i)
            if (slot_[i].state == USED) {
                bool ended = false;
                if (!RT::ok(RT::query(slot_[i].done, ended)))
                    slot_[i].state = LOST;
                else if (ended)
                    return i;
            }
        for (int i = 0; i < N; ++i)
            if (slot_[i].state == NEW) {
                if (RT::ok(RT::create(slot_[i].done))) return i;
                slot_[i].state = LOST;
            }
        return -1;
    }

    std::mutex mu_;
    Slot slot_[N];
};

}  // namespace wnw
