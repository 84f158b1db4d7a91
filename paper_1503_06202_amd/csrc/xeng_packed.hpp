// Interface between the C ABI (xeng_api.cpp) and the packed path: frames
// repacked once into FP6 matrix-core operands (xeng_pack.hip), then correlated
// on 256 x 128 tiles (xcorr_packed.hip).
//
// Packed layout.  The unit is a fragment step: 32 inputs x 32 samples,
// FRAG_BYTES bytes, laid out as the 32 x 32 x 64 FP6 MFMA reads it.  Lane l
// (0..63) holds input l % 32 over the sixteen samples of half l / 32: sixteen
// real codes, then sixteen imaginary codes, six bits each (24 bytes).  The
// first 16 bytes of every lane form the unit's first 1024 bytes, the last 8
// the remaining 512, so that every load of a wave is contiguous.  Units are
// ordered [channel][step][block of 128 inputs][4 fragments].  (Streams of one
// block each, [channel][block][step], made the correlation 2% slower on 2048
// inputs: the workgroups of a channel run in step, and their reads then sit
// whole streams apart.)  A channel has `blocks` blocks (the last one padded)
// and `steps` steps (a multiple of 4: samples are padded to 128 with the code
// of 0 + 0i).
#pragma once

#include "xeng_internal.hpp"

namespace xeng {

constexpr int PK_STEP = 32;                     // samples per fragment step
constexpr int PK_FRAG = 32;                     // inputs per fragment
constexpr int FRAG_BYTES = 64 * 24;             // one unit
constexpr int BLOCK_BYTES = 4 * FRAG_BYTES;     // one step of a block
constexpr int PK_GRAIN = 128;                   // samples per loop round of the kernel
// Samples per block of code sums, which is what one workgroup of the packing
// kernel walks through: 1024 where that gives every compute unit a few
// workgroups, else 256 (a workgroup takes about 1.2 us per 64 samples, one
// after another).  Time slices are whole blocks.
constexpr int PK_SUMB_LONG = 1024, PK_SUMB_SHORT = 256;

struct PackArgs {
  const uint8_t* samples;  // device [T][F][N], channel f0 of the launch at column 0
  const uint8_t* frame_end;  // end of the caller's frame (16-byte reads stay below it)
  int N, nchan;            // inputs; channels of this launch
  int t0, t1;              // samples packed: [t0, t1)
  long long row_stride;    // bytes between time rows (F * N)
  uint8_t* packed;         // device, see above
  int2* sums;              // device [nchan][sum blocks][128 blocks(N)]: real, imaginary codes
  int steps, blocks;       // steps per channel, blocks of 128 inputs
  int nsum, sumb;          // sum blocks per channel, and samples of one
  const int* seg_delay;    // delays per 16 inputs, or NULL
  int dmax;                // the largest delay, to pack by source windows; or -1
  int win;                 // source rows per window, a multiple of 64
};

// Tiles of a channel: per macro row I (256 inputs), its diagonal triangle, then
// the 256 x 128 tiles (I, J), J >= 2 I + 2.
constexpr int PK_PART = 36 * 1024;              // baselines of an item's partial blocks

struct PackedArgs {
  const uint8_t* packed;
  const int2* sums;
  int32_t* vis;            // device, the launch's first channel
  int2* partial;           // device, PK_PART per sliced item, or NULL
  int N, nchan;
  int steps, blocks, nsum, sumb;
  int tiles_per_chan;      // see packed_tiles
  // Head tiles run as nslices slices of slice_len samples, the other (tail)
  // tiles as tail_slices of tail_len; lengths are multiples of sumb (or the
  // whole range).  Sliced tiles (either the head or the tail, not both) store
  // partial blocks, which a second kernel sums.
  int nslices, slice_len, write_mode;
  int head_tiles, tail_slices, tail_len;
};

inline int packed_tiles(int blocks) {
  int t = 0;
  for (int I = 0; 2 * I < blocks; ++I)
    t += 1 + (blocks - 2 * I - 2 > 0 ? blocks - 2 * I - 2 : 0);
  return t;
}

// aligned: N % 16 == 0 and 16-byte aligned rows
hipError_t launch_pack(const PackArgs& a, bool aligned, hipStream_t stream);
hipError_t launch_packed(const PackedArgs& a, hipStream_t stream);
}  // namespace xeng
