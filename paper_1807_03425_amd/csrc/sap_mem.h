// Which of a caller's pointers a kernel may read (host code only).
#pragma once

#include <hip/hip_runtime_api.h>

namespace sap {

// Whether a kernel on `device` can read what the pointer of these attributes
// points at: that device's memory, managed memory, and pinned host memory
// under its own address.  Another device's memory is not among them: a copy
// reads it, a kernel faults unless peer access happens to be on.
inline bool kernel_can_read(const hipPointerAttribute_t &at, int device) {
    switch (at.type) {
        case hipMemoryTypeDevice: return at.device == device;
        case hipMemoryTypeManaged: return true;
        case hipMemoryTypeHost: return at.devicePointer && at.devicePointer == at.hostPointer;
        default: return false;
    }
}

}  // namespace sap
