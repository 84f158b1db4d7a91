// The packed path's first kernel: a frame repacked once into FP6 operands.
//
// A 4-bit code u (0..15) is the FP6 e2m3 number u / 8 as it stands (0..7
// subnormal, 8..15 the first binade), so packing moves bits and converts
// nothing.  A workgroup takes one channel, 128 inputs and one block of code sums (256
// or 1024 samples): it
// stages 64 rows of 128 bytes at a time in LDS as loaded, reads them back
// transposed (see xcorr_tile.hpp), squeezes each lane's sixteen real and
// sixteen imaginary codes from eight to six bits and stores whole fragment
// units.  The per-input code sums (offset corrections) come along, once per
// sample.
//
// Bound by HBM: every sample byte is read once and 1.5 bytes are written, 520
// us for a 1 GiB frame of 2048 inputs, 5.2 TB/s (a plain copy reaches 5.0;
// without the stores 216 us, without the loads 300 us).  Non-temporal loads or
// stores, rows of 256 bytes, two rounds of loads in flight and an XCD-wise
// block order all stayed within 2%.
#include "xcorr_device.hpp"
#include "xeng_packed.hpp"

namespace xeng {

namespace {

constexpr int PK_ROWS = 64;  // rows staged at a time

// Four codes, one a byte, to 24 bits: b0 | b1 << 6 | b2 << 12 | b3 << 18.
__device__ __forceinline__ uint32_t squeeze(uint32_t t) {
  const uint32_t k = 0xF03FF03Fu;
  const uint32_t y = (t & k) | ((t >> 2) & ~k);
  return (y & 0xFFFu) | ((y >> 4) & ~0xFFFu);
}

// Sixteen codes (four words of four) to 96 bits.
__device__ __forceinline__ void squeeze16(const uint32_t (&t)[4], uint32_t (&o)[3]) {
  const uint32_t z0 = squeeze(t[0]), z1 = squeeze(t[1]), z2 = squeeze(t[2]), z3 = squeeze(t[3]);
  o[0] = z0 | (z1 << 24);
  o[1] = (z1 >> 8) | (z2 << 16);
  o[2] = (z2 >> 16) | (z3 << 8);
}

__device__ __forceinline__ v4i load16(const uint8_t* p) {
  v4i v;
  __builtin_memcpy(&v, p, 16);  // any alignment
  return v;
}

// Sixteen sample bytes at any address: one load where all sixteen may be read
// (extra inputs are never written), else the bytes of inputs below N.
__device__ __forceinline__ v4i load_any(const uint8_t* p, bool all, int n0, int N) {
  if (all) return load16(p);
  uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 16; ++e)
    if (n0 + e < N) w[e >> 2] |= (uint32_t)p[e] << (8 * (e & 3));
  return v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
}

// A lane's sixteen samples of one input to its 24 operand bytes, adding their
// codes to sr and sm.
__device__ __forceinline__ void squeeze_step(v2i w0, v2i w1, uint32_t (&o)[6], uint32_t& sr,
                                             uint32_t& sm) {
  const uint32_t w[4] = {(uint32_t)w0.x, (uint32_t)w0.y, (uint32_t)w1.x, (uint32_t)w1.y};
  uint32_t r[4], m[4], x[3], y[3];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    r[e] = (w[e] >> 4) & 0x0F0F0F0Fu;
    m[e] = w[e] & 0x0F0F0F0Fu;
    sr = __builtin_amdgcn_udot4(r[e], 0x01010101u, sr, false);
    sm = __builtin_amdgcn_udot4(m[e], 0x01010101u, sm, false);
  }
  squeeze16(r, x);
  squeeze16(m, y);
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    o[e] = x[e];
    o[3 + e] = y[e];
  }
}

}  // namespace

template <bool ALIGNED, bool SHIFT>
__global__ void __launch_bounds__(256) pack_kernel(PackArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * PK_ROWS * PROW];
  const int b = blockIdx.x;
  const int blk = b % a.blocks, rest = b / a.blocks;
  const int f = rest % a.nchan, sb = rest / a.nchan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int seg = tid & 7, row = tid >> 3;
  const int n0 = blk * BT + 16 * seg;
  const bool whole = n0 + 16 <= a.N;
  const int d = SHIFT && n0 < a.N ? a.seg_delay[n0 >> 4] : 0;
  const uint8_t* col = a.samples + (long long)f * a.N + n0;
  const int step0 = sb * (a.sumb / PK_STEP);
  const int nround = min(a.sumb / PK_STEP, a.steps - step0) / 2;  // 64 rows each

  // one 16-byte piece: inputs n0.. at sample t (of the packed range)
  auto piece = [&](int t) -> v4i {
    const int z = (int)0x88888888u;
    if (n0 >= a.N || t >= a.t1) return v4i{z, z, z, z};
    const uint8_t* p = col + (long long)(t - d) * a.row_stride;
    if (ALIGNED) return *reinterpret_cast<const v4i*>(p);
    // a piece past input N reads into the next channel or row (its extra
    // inputs are never written), but never past the frame
    return load_any(p, whole || p + 16 <= a.frame_end, n0, a.N);
  };
  const int tbase = a.t0 + step0 * PK_STEP + row;
  v4i r0 = piece(tbase), r1 = piece(tbase + 32);
  const int lane_rd = lane_read_offset<FORM_F8>(lane) + 32 * wave;
  uint8_t* out = a.packed +
                 (((long long)f * a.steps + step0) * a.blocks + blk) * BLOCK_BYTES +
                 wave * FRAG_BYTES;
  const long long ostep = (long long)a.blocks * BLOCK_BYTES;
  uint32_t sr = 0u, sm = 0u;
  for (int k = 0; k < nround; ++k) {
    uint8_t* st = lds + (k & 1) * PK_ROWS * PROW;
    *reinterpret_cast<v4i*>(st + row * PROW + 16 * seg) = r0;
    *reinterpret_cast<v4i*>(st + (row + 32) * PROW + 16 * seg) = r1;
    if (k + 1 < nround) {
      r0 = piece(tbase + 64 * (k + 1));
      r1 = piece(tbase + 64 * (k + 1) + 32);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const uint8_t* q = st + lane_rd + PK_STEP * s * PROW;
      const v2i w0 = lds_tr8(q), w1 = lds_tr8(q + 8 * PROW);
      uint32_t o[6];
      squeeze_step(w0, w1, o, sr, sm);
      uint8_t* u = out + (2 * k + s) * ostep;
      *reinterpret_cast<v4i*>(u + 16 * lane) = v4i{(int)o[0], (int)o[1], (int)o[2], (int)o[3]};
      *reinterpret_cast<v2i*>(u + 1024 + 8 * lane) = v2i{(int)o[4], (int)o[5]};
    }
  }
  // the two halves of a step hold the same inputs
  sr += __shfl_xor(sr, 32);
  sm += __shfl_xor(sm, 32);
  if (lane < 32)
    a.sums[((long long)f * a.nsum + sb) * (a.blocks * BT) + blk * BT + 32 * wave + lane] =
        make_int2((int)sr, (int)sm);
}

// The same for delays that differ inside a block of 128 inputs (time
// shifting).  Read by destination, a line's eight groups of 16 inputs come
// from eight rows and every line is fetched eight times (2.08 ms for the GiB
// above with delays of up to 60000 samples); so this kernel walks the source
// instead: a workgroup takes one channel, 128 inputs and `win` source rows,
// reads every line once and hands each group's rows on to its own, shifted
// steps.  Group g's steps start at source rows o_g + 32 k of the window (o_g <
// 32); a step reads up to 32 rows past the window's end.  0.93 ms for that
// frame: 3.0 GB of lines read (the rows of T + D samples) and 1.6 GB written,
// 5.0 TB/s.  LDS holds the last
// two chunks of 64 rows, and a third slot for the next one, so that one
// barrier a chunk suffices.  The code sums are added atomically (two windows
// may meet in a sum block).
template <bool ALIGNED>
__global__ void __launch_bounds__(256) pack_shift_kernel(PackArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[3 * PK_ROWS * PROW];
  const int b = blockIdx.x;
  const int blk = b % a.blocks, rest = b / a.blocks;
  const int f = rest % a.nchan, w = rest / a.nchan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nseg = (a.N + 15) / 16;
  // sample t of the packed range is source row t - d
  const int ws = a.t0 - a.dmax + w * a.win;  // the window's first source row
  const int tend = a.t0 + a.steps * PK_STEP;
  bool any = false;
  for (int k = 8 * blk; k < min(8 * blk + 8, nseg); ++k) {
    const int d = a.seg_delay[k];
    any |= ws + a.win + d > a.t0 && ws + d < tend;
  }
  // the last block's absent groups take delay 0 and read as the code of 0 + 0i
  any |= 8 * blk + 8 > nseg && ws + a.win > a.t0 && ws < tend;
  if (!any) return;  // uniform
  const int seg = tid & 7, row = tid >> 3;
  const int n0 = blk * BT + 16 * seg;
  const bool whole = n0 + 16 <= a.N;
  const int d = n0 < a.N ? a.seg_delay[n0 >> 4] : 0;
  const uint8_t* col = a.samples + (long long)f * a.N + n0;
  auto piece = [&](int r) -> v4i {  // source row r
    const int z = (int)0x88888888u;
    if (n0 >= a.N || r + d < a.t0 || r + d >= a.t1) return v4i{z, z, z, z};
    const uint8_t* p = col + (long long)r * a.row_stride;
    if (ALIGNED) return *reinterpret_cast<const v4i*>(p);
    return load_any(p, whole || p + 16 <= a.frame_end, n0, a.N);
  };
  // this lane's group in the transposed reads: inputs 16 (2 wave + lane / 16 % 2)..
  const int lseg = 8 * blk + 2 * wave + ((lane >> 4) & 1);
  const int ld = lseg < nseg ? a.seg_delay[lseg] : 0;
  const int o = (int)((unsigned)(a.t0 - ld - ws) & 31u);
  const int q0 = (ws + o + ld - a.t0) >> 5;  // the step that starts at row o
  const int lrow = o + 16 * (lane >> 5) + ((lane & 15) >> 1);
  const int lcol = 32 * wave + 16 * ((lane >> 4) & 1) + 8 * (lane & 1);
  const int nchunk = a.win / PK_ROWS;
  const int per_sum = a.sumb / PK_STEP;
  uint8_t* const out = a.packed + (long long)f * a.steps * a.blocks * BLOCK_BYTES +
                       (long long)blk * BLOCK_BYTES + wave * FRAG_BYTES;
  const long long ostep = (long long)a.blocks * BLOCK_BYTES;
  int2* const sums = a.sums + (long long)f * a.nsum * (a.blocks * BT) + blk * BT + 32 * wave + lane;
  uint32_t sr = 0u, sm = 0u;
  v4i r0 = piece(ws + row), r1 = piece(ws + row + 32);
  for (int c = 0; c <= nchunk; ++c) {
    uint8_t* st = lds + (c % 3) * PK_ROWS * PROW;
    *reinterpret_cast<v4i*>(st + row * PROW + 16 * seg) = r0;
    *reinterpret_cast<v4i*>(st + (row + 32) * PROW + 16 * seg) = r1;
    if (c < nchunk) {
      r0 = piece(ws + 64 * (c + 1) + row);
      if (c + 1 < nchunk) r1 = piece(ws + 64 * (c + 1) + row + 32);  // past it: 32 rows
    }
    __syncthreads();
    const int slot0 = (c + 2) % 3 * PK_ROWS;  // rows of chunk c - 1
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if ((c == 0 && u == 0) || (c == nchunk && u == 1)) continue;  // uniform
      const int q = q0 + 2 * c - 1 + u;
      int ra = slot0 + 32 + 32 * u + lrow, rb = ra + 8;
      ra -= ra >= 3 * PK_ROWS ? 3 * PK_ROWS : 0;
      rb -= rb >= 3 * PK_ROWS ? 3 * PK_ROWS : 0;
      const v2i w0 = lds_tr8(lds + ra * PROW + lcol), w1 = lds_tr8(lds + rb * PROW + lcol);
      if (q < 0 || q >= a.steps) continue;  // the same for the 32 lanes of a group
      uint32_t x[6];
      squeeze_step(w0, w1, x, sr, sm);
      uint8_t* d8 = out + q * ostep;
      *reinterpret_cast<v4i*>(d8 + 16 * lane) = v4i{(int)x[0], (int)x[1], (int)x[2], (int)x[3]};
      *reinterpret_cast<v2i*>(d8 + 1024 + 8 * lane) = v2i{(int)x[4], (int)x[5]};
      if ((q + 1) % per_sum == 0 || q + 1 == a.steps || (c == nchunk && u == 0)) {
        const uint32_t tr = sr + __shfl_xor(sr, 32), tm = sm + __shfl_xor(sm, 32);
        if (lane < 32) {
          int* p = &sums[(long long)(q / per_sum) * (a.blocks * BT)].x;
          atomicAdd(p, (int)tr);
          atomicAdd(p + 1, (int)tm);
        }
        sr = sm = 0u;
      }
    }
  }
}

hipError_t launch_pack(const PackArgs& a, bool aligned, hipStream_t stream) {
  if ((a.steps & 3) || a.blocks * BT < a.N ||
      a.sumb % 64 != 0 || a.nsum * (a.sumb / PK_STEP) < a.steps || (long long)a.steps * PK_STEP < a.t1 - a.t0)
    return hipErrorInvalidValue;
  if (a.seg_delay && a.dmax >= 0) {  // by source windows
    if (a.win < 64 || a.win % PK_ROWS != 0) return hipErrorInvalidValue;
    const long long nwin = ((long long)a.steps * PK_STEP + a.dmax + a.win - 1) / a.win;
    const long long grid = (long long)a.blocks * a.nchan * nwin;
    if (grid <= 0) return hipSuccess;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    const hipError_t e = launch_zero(reinterpret_cast<int32_t*>(a.sums),
                                     2LL * a.nchan * a.nsum * a.blocks * BT, stream);
    if (e != hipSuccess) return e;
    if (aligned)
      hipLaunchKernelGGL(pack_shift_kernel<true>, dim3((unsigned)grid), dim3(256), 0, stream, a);
    else
      hipLaunchKernelGGL(pack_shift_kernel<false>, dim3((unsigned)grid), dim3(256), 0, stream, a);
    return hipGetLastError();
  }
  const long long grid = (long long)a.blocks * a.nchan * a.nsum;
  if (grid <= 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 g((unsigned)grid), b(256);
  if (aligned) {
    if (a.seg_delay) hipLaunchKernelGGL((pack_kernel<true, true>), g, b, 0, stream, a);
    else hipLaunchKernelGGL((pack_kernel<true, false>), g, b, 0, stream, a);
  } else {
    if (a.seg_delay) hipLaunchKernelGGL((pack_kernel<false, true>), g, b, 0, stream, a);
    else hipLaunchKernelGGL((pack_kernel<false, false>), g, b, 0, stream, a);
  }
  return hipGetLastError();
}

}  // namespace xeng
