// Second-order forward by a segment walk in fp32 and fp64.  See hla2_walk32.hip.
#pragma once
#include "common.h"

namespace hla {
// d = dv, no decay (masked or unmasked, either input type).
bool walk32_supported(const Fwd& f);
// ws: ws_bytes of device memory; the number of segments is cut to what it holds (one segment needs none).
hipError_t launch_walk32(const Fwd& f, void* ws, size_t ws_bytes, hipStream_t s);
}  // namespace hla
