// Time symmetry of a with-RF waveform (host and device).
#pragma once

#include <stdint.h>

namespace gbs {

// A with-RF waveform that is symmetric in time with one B1 phase: the unit
// normal (nx, ny) of the plane of its fields (compose.hpp); sym = 0: not.
struct WaveSym {
    int32_t sym, pad;
    double nx, ny;
};

}  // namespace gbs
