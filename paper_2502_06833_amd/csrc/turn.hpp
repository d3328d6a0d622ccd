// Whose launch may follow whose: kernels that need the whole chip to themselves.  Host code, no HIP in it.
#pragma once
#include <mutex>

namespace ead {

// Kernels whose workgroups wait for each other (k_decode_stream, k_decode_fused) must all be resident, so two of them must not start side by
// side: each launch first makes its stream wait for the stream the last one on its device went to.  That wait covers the last launch only if
// that launch is queued by then, so the lock is held from the wait until the launch has returned.
template <typename Stream, int DEVICES>
class LaunchTurns {
    struct Turn { const void *holder = nullptr; Stream stream{}; };
    std::mutex m;
    Turn turns[DEVICES];

public:
    // wait(s): the holder's stream waits for what is queued on stream s; launch(): queues the kernel on the holder's.  Both return 0 or an error, which is passed on.
    template <typename Wait, typename Launch>
    auto launch(int device, const void *holder, Stream stream, Wait wait, Launch launch) -> decltype(launch()) {
        std::lock_guard<std::mutex> lock(m);
        Turn &t = turns[device];
        if (t.holder && (t.holder != holder || t.stream != stream))
            if (const auto rc = wait(t.stream)) return rc;
        const auto rc = launch();
        if (!rc) { t.holder = holder; t.stream = stream; }
        return rc;
    }

    // The holder's streams may go away: sync() waits for them, where its launch is the last one.
    template <typename Sync>
    void end(int device, const void *holder, Sync sync) {
        { std::lock_guard<std::mutex> lock(m); if (turns[device].holder != holder) return; }
        sync();
        std::lock_guard<std::mutex> lock(m);
        if (turns[device].holder == holder) turns[device] = Turn{};
    }
};

}  // namespace ead
