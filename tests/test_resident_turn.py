"""Two host threads and the start of one-launch kernels: whoever asks while another thread stands between its question and its
launch has to wait for that launch, and then finds the other stream busy.  A stream that a program made may be gone by the next
call: nothing may be asked of its handle."""
import os
import subprocess

from paper_2605_12245_amd import build

SOURCE = r"""
#include <atomic>
#include <chrono>
#include <cstdio>
#include <thread>
#include "soar_turn.hpp"

struct Fake {
    using Stream = int;
    struct Moment { int stream; };
    using Event = Moment *;
    static constexpr int kMaxDevices = 4;
    static inline std::atomic<bool> running[6], recording[6], gone[6];
    static inline std::atomic<int> dev{0}, touched{0}, made{0};
    static inline bool may_make = true;
    static int device() { return dev; }
    static int capturing(int s) { touched += gone[s]; return recording[s] ? 1 : 0; }
    static bool always_there(int s) { return s == 0; }
    static bool one_per_thread(int s) { return s == 5; }
    static bool busy(int s) { touched += gone[s] || s != 0; return running[s]; }
    static bool make_event(Event &e) { if (may_make) { e = new Moment{-1}; ++made; } return may_make; }
    static bool has_happened(Event e) { return e->stream < 0 || !running[e->stream]; }
};
using Turn = ResidentTurn<Fake>;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

// as a call does: ask, launch if one may
static bool call(int stream, bool *marked = nullptr)
{
    Turn turn;
    if (!turn.take(stream)) return false;
    if (turn.done()) turn.done()->stream = stream;
    if (marked) *marked = turn.done() != nullptr;
    if (!Fake::recording[stream]) Fake::running[stream] = true;
    return true;
}

int main()
{
    std::atomic<bool> asked{false};
    std::thread first([&] {
        Turn turn;
        if (!turn.take(1)) return;
        asked = true;
        std::this_thread::sleep_for(std::chrono::milliseconds(200));
        turn.done()->stream = 1;
        Fake::running[1] = true;                  // the launch
    });
    while (!asked) std::this_thread::yield();
    const bool beside = call(2);
    first.join();
    CHECK(!beside);
    CHECK(call(1));                               // its own stream orders it
    CHECK(!call(2));
    CHECK(!call(0));                              // (a refused call leaves the lock)
    Fake::running[1] = false;
    bool marked;
    CHECK(call(0, &marked) && !marked);           // the default stream: no event, it is asked itself
    CHECK(!call(2));
    Fake::running[0] = false;
    CHECK(call(2, &marked) && marked);
    Fake::recording[3] = true;
    CHECK(call(3, &marked) && !marked);           // recorded only: nothing is held or noted
    Fake::recording[3] = false;
    CHECK(!call(3));
    Fake::gone[2] = true;                         // destroyed, while its launch still runs
    CHECK(!call(1) && !call(0));
    Fake::running[2] = false;
    CHECK(call(1));
    CHECK(Fake::touched == 0);
    Fake::running[1] = false;
    CHECK(call(5));
    CHECK(!call(5));                              // may be another thread's stream
    Fake::running[5] = false;
    CHECK(call(5) && Fake::made == 1);
    Fake::dev = 1;
    Fake::may_make = false;
    CHECK(!call(3) && call(0));                   // no event to be had
    Fake::may_make = true;
    Fake::running[0] = false;
    CHECK(call(3) && call(3) && Fake::made == 2);
    Fake::dev = 4;
    CHECK(!call(0));
    return 0;
}
"""


def test_nobody_starts_between_a_question_and_its_launch(tmp_path):
    src, exe = tmp_path / "turn.cpp", tmp_path / "turn"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", os.path.join(build.HERE, "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
