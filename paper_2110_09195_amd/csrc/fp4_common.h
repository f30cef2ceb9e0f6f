// What the dense FP4 contractions (rows_fp4.hip, conv1x1_fp4.hip) share: buffer resources and the cache policy of their outputs.
#pragma once

#include "snn_internal.h"

namespace snn {

constexpr uint32_t OFF_NONE = 0x80000000u;             // a lane offset past every buffer used here (all < 2 GiB)

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}

// Cache policy of the output's stores: kept in L2 (which merges what two tiles write of one line), non-temporal, or written through L2
// at once (system scope), which leaves nothing to write back at the end of the launch.  store_policy says which.
enum { FP4_STORE_CACHED = 0, FP4_STORE_NT = 1, FP4_STORE_THROUGH = 2 };

// Cache policy of a layer's output in a launch of its own.  A wave stores runs of 32 pixels of a channel plane: whole lines where planes are a
// multiple of 128 bytes, whole half lines of 64, else runs whose ends share a line with another tile.  Measured, us, prepared,
// non-temporal / through / cached (MB of output in brackets):
//   whole lines  64 -> 64 56x56 batch 64 (51) 15.6 / 14.4 / 15.8, batch 128 (103) 24.8 / 27.2 / 27.2, batch 256 42.7 / 47.6 / 51.6
//   half lines   128 -> 128 28x28 batch 128 (51) 19.7 / 18.2 / 18.6, batch 256 (103) 32.0 / 30.0 / 31.3, 256 -> 256 batch 256 (206) 64 / 69 / 70
//   neither      64 -> 512 13x13 batch 256 (89) 40.9 / 34.2 / 22.5, batch 64 (22) 10.4 / 10.6 / 9.7; 100 -> 150 31x31 batch 256 (148)
//                54 / 100 / 48; 512 -> 512 7x7 batch 256 (26) 23.1 / 22.5 / 22.7
//   (runs of whole 16 bytes: 256 -> 256 14x14 batch 64 (13) 10.0 / 9.2 / 9.6, batch 128 (26) 13.9 / 13.3 / 13.9, batch 256 (51) 30.6 / 23.8 / 22.5)
// Written through, runs that share lines are the faster ones only where the last-level cache already holds the output: 256 -> 256 14x14 batch 128 after
// 512 MB of other writes 18.4 / 24.1, batch 64 12.4 / 15.2 (non-temporal / through), so they stay in L2 at every size.
inline int store_policy(const Geom &g, const void *out)
{
    const int64_t mb = (4 * g.P * g.C_out) >> 20;
    const uintptr_t pieces = (uintptr_t)out | (uintptr_t)g.HoWo * 4u;
    if ((pieces & 127) == 0) return mb > 96 ? FP4_STORE_NT : FP4_STORE_THROUGH;
    if ((pieces & 63) == 0) return mb > 144 ? FP4_STORE_NT : FP4_STORE_THROUGH;
    return FP4_STORE_CACHED;
}

}  // namespace snn
