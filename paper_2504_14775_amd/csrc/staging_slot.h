// When a slot of the ring of staging buffers may be written again.  No HIP in here: tests/test_staging_slot.py builds it for the host.
#pragma once

#include <atomic>
#include <chrono>
#include <cstdint>
#include <thread>

// A slot may be written again once the launch that copies it to the device has ended.  A later launch of the batch says so: it stores
// the batch's number in the slot's flag, a word of host memory.
struct StagingSlot {
    enum class State { kFree, kCopied, kFlagged };  // kCopied: no such launch was enqueued (an error came before it)
    State state = State::kFree;
    uint32_t batch = 0;  // number of the batch that used the slot last
};

// Looks at the flag: 64 in a row, then the thread yields; a long wait (batches of milliseconds, three more are queued meanwhile) sleeps
// between them, and from time to time asks for an error of the device.
constexpr int64_t kLooksInARow = 64, kLooksBeforeSleep = 64 * 1024, kLooksBetweenQueries = 1024 * 1024;

// Waits until the slot may be written, however long that takes; returns 0, or the error that ended the wait.  settle() waits for the
// launch of a slot without a flag; error() is asked about once a second whether the flag cannot come any more.
template <class Settle, class Error>
int await_staging_slot(StagingSlot& slot, const volatile uint32_t* flag, Settle settle, Error error) {
    if (slot.state == StagingSlot::State::kCopied) {
        if (const int e = settle()) return e;
    } else if (slot.state == StagingSlot::State::kFlagged) {
        for (int64_t n = 1; *flag != slot.batch; ++n) {
            if (n % kLooksInARow != 0) continue;
            if (n < kLooksBeforeSleep) std::this_thread::yield();
            else std::this_thread::sleep_for(std::chrono::microseconds(20));
            if (n % kLooksBetweenQueries != 0) continue;
            if (const int e = error()) return e;
        }
        std::atomic_thread_fence(std::memory_order_acquire);
    }
    slot.state = StagingSlot::State::kFree;
    return 0;
}
