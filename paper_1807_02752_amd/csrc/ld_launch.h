// ld_launch.h -- what the host decides before a launch, without HIP types: the dynamic LDS that
// a kernel has been granted.  Not part of the C ABI.
#pragma once

#include <atomic>
#include <cstddef>
#include <mutex>

constexpr int kMaxDevices = 64;

// The dynamic LDS granted to one kernel on each GPU.
struct LdsGrants {
    std::mutex mu;
    std::atomic<size_t> bytes[kMaxDevices] = {};
};

// Raises the dynamic LDS limit of Kernel on `device` to `bytes` by set(), which says whether that
// worked, unless it is there already.  The record is the kernel's own (a template argument: two
// instantiations of one kernel template have the same type) and the GPU's, and set() runs under
// its lock, so that no thread lowers what another has just raised.
template <auto Kernel, typename Set>
void raise_lds(int device, size_t bytes, Set set) {
    static LdsGrants grants;
    if (device < 0 || device >= kMaxDevices) {
        (void)set();
        return;
    }
    std::atomic<size_t>& have = grants.bytes[device];
    if (bytes <= have.load(std::memory_order_acquire)) return;
    std::lock_guard<std::mutex> lock(grants.mu);
    if (bytes > have.load(std::memory_order_relaxed) && set()) have.store(bytes, std::memory_order_release);
}
