// Which host thread may start a one-launch kernel.
#pragma once
#include <mutex>

namespace {

// Two one-launch kernels that start at the same time on two streams can each take part of the compute
// units and then wait for the rest in vain (until the bounded wait gives up).  Calls on one stream are
// ordered by the stream.  For calls that arrive on a different stream than the one-launch kernel before
// them, this asks whether that earlier stream has drained; if it has not (or the question cannot be asked:
// either stream is being captured into a graph), the caller takes the path of several launches for this call.
// The lock is held until the caller has launched: a thread that asks between another's question and its launch would
// find that stream empty and start beside it.
// A stream that a program made may be gone when the next call arrives, and a handle of it may not be asked anything: its launches leave an
// event behind, which is this library's own (launches of an empty kernel back to back: 2.5 us each, with the event attached to the launch 4.0,
// recorded behind it 5.0).  The null stream is always there, and is asked itself.
// Best effort: replays of captured graphs and other processes on the same GPU are not seen here; the
// bounded wait and SOAR_STATUS_GAVE_UP cover those.
//
// Gpu: Stream, Event (pointers), kMaxDevices, device() (-1: unknown), capturing(stream) (negative: cannot be asked), always_there(stream),
// one_per_thread(stream): a handle that is another stream in every thread, busy(stream), make_event(event), has_happened(event)
template <typename Gpu>
class ResidentTurn {
    struct Last {
        std::mutex mu;
        typename Gpu::Stream stream{};
        typename Gpu::Event launched{};
        bool any = false;
    };
    std::unique_lock<std::mutex> hold;
    typename Gpu::Event mark{};

public:
    // true: launch on `st` while this object lives, with done() as the event that the launch completes, if there is one
    bool take(typename Gpu::Stream st)
    {
        static Last last[Gpu::kMaxDevices];
        const int dev = Gpu::device();
        if (dev < 0 || dev >= Gpu::kMaxDevices) return false;
        const int capturing = Gpu::capturing(st);
        if (capturing != 0) return capturing > 0;                // recorded, not started: nothing to track
        Last &before = last[dev];
        std::unique_lock<std::mutex> lock(before.mu);
        if (before.any && (before.stream != st || Gpu::one_per_thread(st))) {
            // may still be running: do not start beside it
            if (Gpu::always_there(before.stream) ? Gpu::busy(before.stream) : !Gpu::has_happened(before.launched)) return false;
        }
        if (!Gpu::always_there(st)) {
            if (!before.launched && !Gpu::make_event(before.launched)) return false;
            mark = before.launched;
        }
        before.stream = st;
        before.any = true;
        hold = std::move(lock);
        return true;
    }
    typename Gpu::Event done() const { return mark; }
};

}  // namespace
