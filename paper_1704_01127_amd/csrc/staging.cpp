#include "staging.h"

#include <cstring>
#include <mutex>
#include <vector>

namespace qsim {
namespace {

// Blocks a device's pool may hold (1 MiB of pinned memory in all). They are
// kept for the next call until the process ends: allocating one takes longer
// than the copy it saves, and freeing one waits for the device.
constexpr int kStageBlocks = 8;

std::mutex g_mu;
std::vector<StageBlock*> g_blocks;  // of every device, least recently used first

bool idle(const StageBlock& b) {
    if (b.taken) return false;
    for (int i = 0; i < b.n_flags; ++i)
        if (__atomic_load_n(b.flags() + i, __ATOMIC_ACQUIRE) != b.seq) return false;
    return true;
}

// hipHostMalloc while another thread captures a graph would end that capture
// unless this thread opts out of it.
bool allocate(StageBlock* b) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    void *h = nullptr, *d = nullptr;
    const size_t bytes = kStageBytes + kStageFlags * sizeof(uint32_t);
    bool ok = hipHostMalloc(&h, bytes, hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess;
    if (ok && hipHostGetDevicePointer(&d, h, 0) != hipSuccess) {
        (void)hipHostFree(h);
        ok = false;
    }
    if (!ok) (void)hipGetLastError();
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (!ok) return false;
    std::memset(h, 0, bytes);
    b->host = static_cast<char*>(h);
    b->dev = static_cast<char*>(d);
    return true;
}

}  // namespace

StageBlock* stage_acquire(hipStream_t st) try {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (cs != hipStreamCaptureStatusNone) return nullptr;
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_mu);
    int have = 0;
    StageBlock* b = nullptr;
    for (size_t i = 0; i < g_blocks.size(); ++i) {
        if (g_blocks[i]->device != device) continue;
        ++have;
        if (!idle(*g_blocks[i])) continue;
        b = g_blocks[i];
        g_blocks.erase(g_blocks.begin() + i);
        g_blocks.push_back(b);
        break;
    }
    if (!b) {
        if (have >= kStageBlocks) return nullptr;
        b = new StageBlock;
        b->device = device;
        if (!allocate(b)) {
            delete b;
            return nullptr;
        }
        g_blocks.push_back(b);
    }
    b->taken = true;
    b->n_flags = 0;
    ++b->seq;
    return b;
} catch (...) {  // no memory for the bookkeeping
    return nullptr;
}

void stage_release(StageBlock* b, int n_flags) {
    std::lock_guard<std::mutex> lock(g_mu);
    b->n_flags = n_flags;
    b->taken = false;
}

}  // namespace qsim
