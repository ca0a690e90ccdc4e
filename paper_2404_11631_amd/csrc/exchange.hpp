// exchange.hpp -- values passed between the workgroups of one cooperative launch.
//
// A chain of dependent launches costs ~2.7 us per launch on gfx950 before any work; the iterations
// of the single-replication paths are such chains. Inside one launch a workgroup publishes a value
// as one 64-bit word, the value in the high half and the iteration's tag in the low one, stored and
// loaded with relaxed agent-scope atomics: a reader that sees the tag has the value of the same
// store, so no fence is needed (a release fence writes back the whole L2 of an XCD, which made a
// counter-based form five times slower than the launches it replaced), and the reader's poll is the
// only wait. Slots alternate between two buffers by the iteration's parity, each workgroup's on a 64-byte line
// of its own; a workgroup publishes
// iteration t + 1 only after it has read every value of iteration t, so a slot is overwritten (at
// t + 2) only after all have read it.
//
// Every wait is bounded: a poll that does not see its tag within kPollLimit rounds (seconds, where a
// value arrives within microseconds) gives up, the workgroup raises the run's failure word and
// leaves, and the others follow by their own limits; the host reports the failure or runs the
// launch-by-launch form. The launches are cooperative, so all workgroups are resident together.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fw {

constexpr uint32_t kPollLimit = 1u << 22;

__device__ __forceinline__ void exchange_put(uint64_t *slot, uint32_t value, uint32_t tag)
{
    __hip_atomic_store(slot, (static_cast<uint64_t>(value) << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t exchange_get(const uint64_t *slot)
{
    return __hip_atomic_load(const_cast<uint64_t *>(slot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t failure_get(const uint32_t *fail)
{
    return __hip_atomic_load(const_cast<uint32_t *>(fail), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void failure_raise(uint32_t *fail)
{
    __hip_atomic_store(fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace fw
