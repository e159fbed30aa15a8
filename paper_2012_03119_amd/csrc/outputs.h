// Where a call's output lies, host only.
#pragma once

#include <cstdint>

namespace gss {

struct OutputPlace {
    bool device = false;   // device memory (not managed, not host)
    int ordinal = -1;      // its device
    uintptr_t address = 0;
};

// Whether a kernel on `device` may store 8-byte words there itself.  Another device's
// memory is reached by a copy only: peer access need not be enabled.
inline bool stores_directly(const OutputPlace &p, int device) {
    return p.device && p.ordinal == device && (p.address & 7) == 0;
}

}  // namespace gss
