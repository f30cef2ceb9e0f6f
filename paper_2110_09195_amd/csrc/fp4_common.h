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
// at once (device scope), which leaves nothing to write back at the end of the launch.  store_policy says which.
enum { FP4_STORE_CACHED = 0, FP4_STORE_NT = 1, FP4_STORE_THROUGH = 2 };
constexpr int AUX_CACHED = 0, AUX_NT = 2 /* nt */, AUX_THROUGH = 16 /* sc1 */;      // the store instruction's operand for each

// Cache policy of a layer's output in a launch of its own.  A wave stores runs of 32 pixels of a channel plane: whole lines where planes are a
// multiple of 128 bytes, whole half lines of 64, else runs whose ends share a line with another tile.  Measured, us, prepared, cached /
// non-temporal / through, warm (three outputs in turn), then after 512 MB of other writes (which leave the last-level cache full; with the
// two events' share), MB of output in brackets:
//   whole lines  16 -> 16 32x32 batch 256 (16) 8.1 / 6.8 / 6.0, 10.8 / 9.4 / 8.8; 64 -> 64 56x56 batch 32 (24) 9.2 / 8.8 / 7.8, 12.2 / 11.7 / 10.8,
//                batch 64 (49) 15.7 / 14.9 / 13.9, 19.2 / 17.7 / 18.0, batch 128 (98) 26.6 / 23.7 / 24.1, 29.0 / 28.2 / 28.3,
//                batch 256 (196) 49.6 / 40.9 / 43.2, 52.1 / 51.5 / 51.7
//   half lines   128 -> 128 28x28 batch 64 (24) 10.3 / 9.8 / 8.5, 13.5 / 12.8 / 11.9, batch 128 (49) 17.5 / 18.3 / 15.7, 21.4 / 20.8 / 20.1,
//                batch 256 (98) 29.7 / 29.5 / 27.8, 32.6 / 33.6 / 32.1; 256 -> 256 28x28 batch 256 (206) warm 70 / 64 / 69
//   neither      256 -> 256 14x14 batch 32 (6) 6.9 / 7.3 / 6.8, 10.4 / 10.2 / 11.4, batch 64 (12) 9.2 / 9.0 / 8.5, 12.8 / 12.0 / 15.2, batch 128 (24)
//                13.0 / 13.6 / 12.4, 16.8 / 17.2 / 24.1, batch 256 (49) 20.3 / 29.8 / 21.9, 25.1 / 29.4 / 39.3; 64 -> 512 13x13 batch 64 (21)
//                9.4 / 10.2 / 10.2, 13.1 / 13.2 / 20.6, batch 256 (84) 21.6 / 39.5 / 39.1, 27.5 / 41.2 / 59.7; 100 -> 150 31x31 batch 256 (141)
//                46.7 / 53.4 / 100.8, 49.3 / 55.2 / 106.6
// Written to memory (WRITE_SIZE, MiB, in the same order): half lines, batch 128 (49.0) 49.1 / 53.7 / 49.0; neither, 256 -> 256 batch 128 (24.5) 24.6 / 26.2 /
// 28.0, 64 -> 512 batch 256 (84.5) 85.7 / 109.0 / 106.4: lines that two tiles share are written once from L2.
// Runs that share lines stay in L2 at every size: through is up to a tenth faster warm and half as slow again after other writes.  Non-temporal
// is the faster one of two after other writes up to some 18 MB, by 1 to 9 % (at the 9 to 18 MB that fill part of L2 most), and warm
// there on some cards (12 MB above, by 2 %) but not on others (the same layer 9.0 / 9.5, 128 -> 300 7.3 / 7.9, 1x1 256 -> 1024 6.1 / 7.0).
inline int store_policy(const Geom &g, const void *out)
{
    const int64_t mb = (4 * g.P * g.C_out) >> 20;
    const uintptr_t pieces = (uintptr_t)out | (uintptr_t)g.HoWo * 4u;
    if ((pieces & 127) == 0) return mb > 96 ? FP4_STORE_NT : FP4_STORE_THROUGH;
    if ((pieces & 63) == 0) return mb > 144 ? FP4_STORE_NT : FP4_STORE_THROUGH;
    return FP4_STORE_CACHED;
}

}  // namespace snn
