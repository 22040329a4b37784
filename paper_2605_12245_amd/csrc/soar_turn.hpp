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
// Best effort: replays of captured graphs and other processes on the same GPU are not seen here; the
// bounded wait and SOAR_STATUS_GAVE_UP cover those.
//
// Gpu: `Stream`, kMaxDevices, device() (-1: unknown), capturing(stream) (negative: no such stream), busy(stream)
template <typename Gpu>
class ResidentTurn {
    struct Last {
        std::mutex mu;
        typename Gpu::Stream stream{};
        bool any = false;
    };
    std::unique_lock<std::mutex> hold;

public:
    // true: launch on `st` while this object lives
    bool take(typename Gpu::Stream st)
    {
        static Last last[Gpu::kMaxDevices];
        const int dev = Gpu::device();
        if (dev < 0 || dev >= Gpu::kMaxDevices) return false;
        const int capturing = Gpu::capturing(st);
        if (capturing != 0) return capturing > 0;                // recorded, not started: nothing to track
        Last &before = last[dev];
        std::unique_lock<std::mutex> lock(before.mu);
        if (before.any && before.stream != st) {
            const int that = Gpu::capturing(before.stream);
            if (that > 0) return false;                          // a query would break that capture
            if (that == 0 && Gpu::busy(before.stream)) return false;      // may still be running: do not start beside it
            // (a stream that no longer exists has nothing in flight)
        }
        before.stream = st;
        before.any = true;
        hold = std::move(lock);
        return true;
    }
};

}  // namespace
