"""CPU test of the rule by which key-sensitivity launches share the library's scratch slots
(csrc/wnw_slots.h), against a model of streams and events: a launch waits for no other stream, and two
launches that may run at once never hold one slot."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MODEL = r"""
#include "wnw_slots.h"

#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>

#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

// A stream is a counter of work done and enqueued; an event is a point of a stream.
struct Stream { long done = 0, end = 0; };
struct Ev { int stream = -1; long at = 0; };
static std::map<int, Stream> S;
static std::vector<Ev> E;
static int cross_waits = 0, queries = 0;
static bool events_gone = false, record_fails = false, create_fails = false;

struct RT {
    using Stream = int;
    using Event = int;
    using Error = int;
    static bool ok(int e) { return e == 0; }
    static int create(int &e) { if (create_fails) return 1; e = (int)E.size(); E.emplace_back(); return 0; }
    static int query(int e, bool &ended)
    {
        ++queries;
        if (events_gone) return 1;
        ended = E[e].stream < 0 || S[E[e].stream].done >= E[e].at;
        return 0;
    }
    static int wait(int st, int e)
    {
        if (events_gone) return 1;
        if (E[e].stream != st) ++cross_waits;
        return 0;
    }
    static int record(int e, int st) { if (record_fails) return 1; E[e] = {st, S[st].end}; return 0; }
    static bool shared_handle(int st) { return st == 2; }
};

constexpr int N = 8;
struct User { int stream = -1; long at = 0; };
static User user[N];

// One launch on a stream; false: not split.  Aborts when the slot may be in use by another stream.
template <class P>
static bool launch(P &pool, int st, int &err)
{
    return pool.run(st, err, [&](int i) {
        if (user[i].stream >= 0 && (user[i].stream != st || st == 2) && S[user[i].stream].done < user[i].at) {
            std::printf("slot %d of stream %d given to stream %d\n", i, user[i].stream, st);
            std::exit(1);
        }
        user[i] = {st, ++S[st].end};
        return 0;
    });
}

int main()
{
    int err = 0;
    {   // a stream that is held back, then many calls on another: none waits, all are split
        SlotPoolT pool;
        CHECK(launch(pool, 10, err) && err == 0);
        for (int i = 0; i < 100; ++i) CHECK(launch(pool, 11, err) && err == 0);
        CHECK(cross_waits == 0);
        // more streams than slots, nothing done yet: the first seven get one, the others none
        int split = 0;
        for (int s = 12; s < 30; ++s) split += launch(pool, s, err);
        CHECK(split == N - 2 && cross_waits == 0);
        // once one has ended, its slot serves any stream
        S[13].done = S[13].end;
        CHECK(launch(pool, 29, err) && !launch(pool, 28, err) && cross_waits == 0);
    }
    for (auto &u : user) u = {};
    {   // one handle value for several streams (per-thread default streams): their order is unknown
        SlotPoolT pool;
        int split = 0;
        for (int i = 0; i < 20; ++i) split += launch(pool, 2, err);
        CHECK(split == N);
        S[2].done = S[2].end;
        CHECK(launch(pool, 2, err));
    }
    for (auto &u : user) u = {};
    {   // random streams and progress
        SlotPoolT pool;
        std::srand(1);
        for (int i = 0; i < 200000; ++i) {
            const int s = 40 + std::rand() % 12;
            if (std::rand() % 3)
                launch(pool, s, err);
            else
                S[s].done += std::rand() % (S[s].end - S[s].done + 1);
            CHECK(err == 0);
        }
        CHECK(cross_waits == 0);
    }
    for (auto &u : user) u = {};
    {   // events that a device reset took away, an event that cannot be recorded or created: never an unsafe
        // slot, and no error for what can be computed unsplit
        SlotPoolT pool;
        CHECK(launch(pool, 60, err));
        events_gone = true;
        for (int i = 0; i < 3; ++i) launch(pool, 60, err), launch(pool, 61, err);
        CHECK(err == 0);
        events_gone = false;
        SlotPoolT lost;
        for (auto &u : user) u = {};
        record_fails = true;
        CHECK(launch(lost, 62, err) && err != 0);
        record_fails = false;
        for (int i = 0; i < 50; ++i) {
            CHECK(launch(lost, 62, err) && err == 0 && user[0].stream == 62 && user[0].at == 1);
        }
        SlotPoolT none;
        create_fails = true;
        CHECK(!launch(none, 63, err));
    }
    std::printf("ok %d queries\n", queries);
    return 0;
}
"""


def test_slots_wait_for_no_other_stream(tmp_path):
    src, exe = tmp_path / "slots.cpp", tmp_path / "slots"
    src.write_text(MODEL.replace("int main()", "using SlotPoolT = wnw::SlotPool<RT, N>;\n\nint main()"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2608_22704_amd", "csrc"), str(src), "-o", str(exe), "-lpthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
