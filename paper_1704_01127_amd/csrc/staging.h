// Pinned host blocks through which descriptors reach the device and sums come
// back: the matrix builder reads a block directly and the final reduction
// writes one, so a call needs no copy and the host does not wait for its
// descriptors to be read.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace qsim {

// A block's data area, and the words in which the work-groups that read it
// mark their end.
constexpr size_t kStageBytes = size_t(128) << 10;
constexpr int kStageFlags = 1024;

struct StageBlock {
    char* host = nullptr;    // kStageBytes of data, then kStageFlags words
    char* dev = nullptr;     // the same memory as the device sees it
    uint32_t seq = 0;        // value of the flags when the block's last reader has ended
    int n_flags = 0;         // how many work-groups read it last
    int device = -1;
    bool taken = false;      // between acquire and release
    uint32_t* flags() const { return reinterpret_cast<uint32_t*>(host + kStageBytes); }
    uint32_t* dev_flags() const { return reinterpret_cast<uint32_t*>(dev + kStageBytes); }
};

// A free block of the current device, or null: where `st` is being captured
// (the graph would read the block again on a replay), when every block of the
// bounded pool is still being read, or when pinned memory is short. The caller
// then copies from pageable memory. Safe from any thread.
StageBlock* stage_acquire(hipStream_t st);

// Give a block back. `n_flags` work-groups of the launches just enqueued read
// it and store its seq in the first n_flags flags when they end (0: the work
// that used the block is known to have ended).
void stage_release(StageBlock* b, int n_flags);

}  // namespace qsim
