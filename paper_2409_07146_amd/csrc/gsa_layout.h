// Layout descriptor of the per-chunk memory snapshots kept in the workspace.
#pragma once
#include <hip/hip_runtime.h>

namespace gsa {

// A snapshot of the joint memory [Kt | Vt] (or of its gradient) is one record per (chunk, head)
// or per (sequence, head): the key part followed by the value part.  Each part is stored as
// tiles of kSnapTile columns, tile after tile, every tile [m][kSnapTile] with the column
// fastest: element (slot i, column c) of a part sits at
//     (c / kSnapTile) * m * kSnapTile + i * kSnapTile + c % kSnapTile.
// A scan workgroup owns one tile and writes it as one contiguous block (rows of a [m][d] array
// would be 128-byte pieces a kilobyte apart, which the memory system serves measurably slower);
// a contraction over the head dimension still finds 8 consecutive columns of a slot in one
// 16-byte piece, and the apply kernel, which contracts over the slots, transposes the column
// slice it needs on its way into LDS.  Offsets are in elements from the start of the record.
constexpr int kSnapTile = 64;

// The lanes of a wave load up to this many consecutive rows of a token tensor (a row: all heads of a token) at 32-bit byte offsets
// from the first.  The host refuses rows so long that they would wrap (H * d from 153 million in fp32, 306 million in bf16).
constexpr int kLaneRows = 8;

// Chunks per segment when the scans cut long sequences into segments.
constexpr int kSegChunks = 32;

// When a scan walks its sequences whole although they could be cut into segments.  longest: chunks of the longest sequence,
// steps: chunks times workgroups per chunk (heads and column slices).  In one walk the launch waits for the chain of the
// longest sequence, or for all steps where they fill the chip; in segments for two chains of kSegChunks chunks and what is
// around them, or for all steps twice, since the tokens are read twice.  Time of the forward call, whole / in segments, us:
//   the chain (1 head, d = 64)      56 chunks     66          84
//     bf16  16 slots                  33 / 38       36 / 38     42 / 38
//           64                        48 / 54       54 / 55     63 / 55
//          128                        68 / 71       76 / 73     89 / 74
//     fp32  16                        44 / 50       49 / 50     57 / 50
//           64                        82 / 85       92 / 87    110 / 86
//          128                       132 / 133     153 / 136   188 / 135
//   all steps (n equal sequences, 4 heads, d = 512, 64 slots; steps per chunk of the longest: 64 n)
//     bf16  n = 1    72 chunks 87 / 87, 144 151 / 130;  n = 2    72 116 / 146, 256 347 / 366;  n = 4    144 308 / 403
//     fp32  n = 1    72 chunks 147 / 141, 144 239 / 173;  n = 2    72 177 / 200, 96 218 / 218, 144 333 / 304;  n = 4    144 482 / 569
// (fp32 with 128 slots as with 64; with 16 and 32 as bf16.)
__host__ __device__ inline bool scan_unsegmented(bool f32, int m, long long longest, long long steps)
{
    const int few = f32 ? (m > 16 ? 64 : 68) : m > 64 ? 64 : m > 32 ? 68 : 72;
    long long wide = steps / 110;
    if (f32 && m > 32) {
        wide = wide < 96 ? wide : 96;
        wide = wide > steps / 160 ? wide : steps / 160;
    }
    return longest <= (wide > few ? wide : few);
}

// The device kernels take the read-out and the feature-map switch in one int: the Readout value in
// the low byte, this bit for "q, k, v are raw projections: apply the feature map to them".
constexpr int kFeatureMapBit = 0x100;
constexpr int kReadoutMask = 0xff;

struct StateLayout {
    long long stride;   // elements per record
    long long oK, oV;   // key part, value part
};

// Offset of columns k0 .. k0+7 (k0 % 8 == 0) of slot 0 inside a part with m slots.
template <int M> __device__ __forceinline__ unsigned snap_col(int k0)
{
    return (unsigned)(k0 / kSnapTile) * (unsigned)(M * kSnapTile) + (unsigned)(k0 % kSnapTile);
}

}  // namespace gsa
