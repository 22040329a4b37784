"""Two host threads and the start of one-launch kernels: whoever asks while another thread stands between its question and its
launch has to wait for that launch, and then finds the other stream busy."""
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
    static constexpr int kMaxDevices = 2;
    static inline std::atomic<bool> running[4], recording[4], gone[4];
    static inline std::atomic<int> dev{0};
    static int device() { return dev; }
    static int capturing(int s) { return gone[s] ? -1 : recording[s] ? 1 : 0; }
    static bool busy(int s) { return running[s]; }
};
using Turn = ResidentTurn<Fake>;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main()
{
    std::atomic<bool> asked{false};
    std::thread first([&] {
        Turn turn;
        if (!turn.take(1)) return;
        asked = true;
        std::this_thread::sleep_for(std::chrono::milliseconds(200));
        Fake::running[1] = true;                  // the launch
    });
    while (!asked) std::this_thread::yield();
    bool beside;
    { Turn turn; beside = turn.take(2); }
    first.join();
    CHECK(!beside);
    { Turn turn; CHECK(turn.take(1)); }           // its own stream orders it
    { Turn turn; CHECK(!turn.take(2)); }
    { Turn turn; CHECK(!turn.take(2)); }          // (a refused call leaves the lock)
    Fake::running[1] = false;
    { Turn turn; CHECK(turn.take(2)); }
    Fake::running[2] = true;
    Fake::recording[3] = true;
    { Turn turn; CHECK(turn.take(3)); Turn other; CHECK(!other.take(1)); }      // recorded only: nothing is held or noted
    Fake::recording[2] = true;
    { Turn turn; CHECK(!turn.take(1)); }
    Fake::recording[2] = false;
    Fake::gone[2] = true;
    { Turn turn; CHECK(turn.take(1)); }           // the stream before is gone
    { Turn turn; CHECK(!turn.take(2)); }
    Fake::running[1] = true;
    Fake::dev = 1;
    { Turn turn; CHECK(turn.take(3) && turn.take(0)); }
    Fake::dev = 2;
    { Turn turn; CHECK(!turn.take(0)); }
    return 0;
}
"""


def test_nobody_starts_between_a_question_and_its_launch(tmp_path):
    src, exe = tmp_path / "turn.cpp", tmp_path / "turn"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", os.path.join(build.HERE, "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
