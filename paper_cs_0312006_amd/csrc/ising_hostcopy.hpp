// Copies from device memory to ordinary (pageable) host memory, for the
// calls that hand whole lattices and maps to the caller.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace ising {

// Pinned stages are shared by all contexts of the process: at most
// kMaxStages of kStageBytes exist (copies beyond them use the runtime's own
// path), and they are freed when the last context is destroyed. Every context
// holds one reference from its creation to its destruction.
void hostcopy_retain();
void hostcopy_release();

// Copy `bytes` from device memory src (on the current device) to host memory
// dst after the earlier work of stream s, and wait for it. Safe to call from
// several threads. dst need not be pinned; where it is, the copy is direct.
hipError_t copy_to_host(void* dst, const void* src, size_t bytes, hipStream_t s);

}  // namespace ising
