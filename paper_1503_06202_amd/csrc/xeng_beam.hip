// Discrete beamforming (Sec. IV-C, "Discrete Beamforming"): the data of all
// inputs are phase-shifted and summed so that a signal from one direction adds
// in phase, and the sum is written out at the sample cadence:
//
//     y[t][f][b] = sum_n w[f][b][n] x[t][f][n]      (complex, no conjugate)
//
// Per channel this is one real int8 contraction on the matrix cores,
//
//     Y (T x 2B) = U (T x 2N) . Wop (2N x 2B) - 8 . 1 colsum(Wop),
//
// where U holds the offset-binary codes u = v + 8 (0..15) of the real and
// imaginary parts of every input, column 2b + 0 of Wop holds (w_re, -w_im) and
// column 2b + 1 holds (w_im, w_re) against (u_re, u_im), and the last term,
// 8 sum_k Wop[k][c], removes the offsets exactly.
//
// The path is bound by HBM: every sample byte is read once (N bytes per time
// and channel) while the output is 8B bytes.  A workgroup takes one channel
// and NW x TT x 32 consecutive times; consecutive workgroups take consecutive
// channels of the same times, so that together they read whole time rows of
// the frame.  Each wave streams its TT tiles of 32 times straight from global
// memory, 128 inputs (128 bytes of every row) per step with the next step's
// loads in flight.  The weight operands, prepared once per plan in the MFMA lane
// order, are staged per step into LDS by the whole workgroup (double
// buffered, one barrier per step), so that its waves read them once from
// L2 between them.  A lane's A operand for one MFMA is 8 inputs of one time:
// 8 real codes, then 8 imaginary codes; in step s, k-step q (0..7), lane half
// h holds inputs 128 s + 32 (q >> 1) + 16 h + 8 (q & 1) + 0..7.
//
// Three or four component tiles: with one time tile a wave reads a weight
// operand from LDS for every MFMA and a workgroup reads all weights of its
// channel (N x 8B bytes, a quarter of a frame's traffic at N = 2048, B = 64) for
// 128 rows; two time tiles and eight waves halve the first and quarter the
// second.  Five or six tiles leave registers for one time tile a wave, and one
// launch that reads the samples once.
//
// Output rows (8B bytes) are stored tile by tile within a row, past the caches
// where rows are whole sectors: with the row's tiles apart in time, lines left
// L2 in pieces.
//
// Measured, us, before -> after (bytes at 5.0 TB/s):
//   N = 2048, F = 16, T = 32768   B = 16 236 -> 229 (228), B = 64 500 -> 366
//                                 (268), B = 96 798 -> 598 (295)
//   N = 64, F = 64, T = 16384, B = 40     182 -> 92 (81)
//   N = 1090, F = 8, T = 20011, B = 20    375 -> 81 (40), byte loads before
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "xcorr_tile.hpp"
#include "xeng_internal.hpp"

namespace xeng {
namespace {

constexpr unsigned kLow4 = 0x0F0F0F0Fu;

// Operand of k-step q (0..7) from the lane's 64 sample bytes of one step.
__device__ __forceinline__ v4i a_operand(const v4i (&raw)[4], int q) {
  const uint32_t w0 = (uint32_t)raw[q >> 1][2 * (q & 1)];
  const uint32_t w1 = (uint32_t)raw[q >> 1][2 * (q & 1) + 1];
  return v4i{(int)((w0 >> 4) & kLow4), (int)((w1 >> 4) & kLow4), (int)(w0 & kLow4),
             (int)(w1 & kLow4)};
}

// The lane's 64 sample bytes of one time and step: bytes 32 i + 16 h .. + 15
// of the step, i = 0..3 (off includes 16 h).  Aligned rows take 16-byte buffer
// loads, which read 0 past the frame; others take 16-byte loads at any address
// (full rate on gfx950) unless the wave's step reaches past the frame's last
// byte, at nrec.
template <bool ALIGNED>
__device__ __forceinline__ void load_step(v4i (&raw)[4], __amdgpu_buffer_rsrc_t rs,
                                          const uint8_t* __restrict__ base, int off, int nrec) {
  if (ALIGNED) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      raw[i] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 32 * i, 0, 0));
  } else if (__all(off + 112 <= nrec)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) __builtin_memcpy(&raw[i], base + (uint32_t)off + 32 * i, 16);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          w |= (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs, off + 32 * i + 4 * d + e, 0, 0)
               << (8 * e);
        raw[i][d] = (int)w;
      }
  }
}

// NB: beam-component tiles (32 columns of Y each) of this launch; TT: time tiles
// of 32 per wave; NW: waves.
template <int NB, int TT, int NW, bool ALIGNED>
__global__ void __launch_bounds__(64 * NW) beam_kernel(BeamArgs a) {
  constexpr int WT = 512 * NB / (64 * NW);  // weight operands a thread stages
  __shared__ __attribute__((aligned(16))) v4i wl[2][8][NB][64];  // a step's weights, twice
  const int logical = xcd_logical_id(blockIdx.x, gridDim.x);
  const int f = logical % a.F;
  const int tb = logical / a.F;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h = lane >> 5, r = lane & 31;
  const int tbase = (tb * NW + wave) * TT * 32;
  const long long row_stride = (long long)a.F * a.N;
  // bytes from this channel's first sample to the end of the launch's frame
  const int nrec = (int)((long long)a.T * row_stride - (long long)f * a.N);
  const uint8_t* const base = a.samples + (long long)f * a.N;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, nrec, 0x00020000);
  const v4i* __restrict__ wop = reinterpret_cast<const v4i*>(a.wop);

  int off[TT];
#pragma unroll
  for (int j = 0; j < TT; ++j)
    off[j] = (int)((ALIGNED ? tbase + 32 * j + r : min(tbase + 32 * j + r, a.T - 1)) * row_stride) +
             16 * h;
  // A step's weights are 8 x NB x 64 operands; thread tid stages operands
  // e = tid + 64 NW k, k < WT, with e = (q NB + c) 64 + lane.
  auto wsrc = [&](int s, int e) {
    const int l = e & 63, c = (e >> 6) % NB, q = (e >> 6) / NB;
    return wop[((((long long)f * a.S + s) * 8 + q) * a.NBT + a.c0 + c) * 64 + l];
  };
  v4i* const wflat0 = &wl[0][0][0][0];
  v4i* const wflat1 = &wl[1][0][0][0];

  v16i acc[TT][NB];
#pragma unroll
  for (int j = 0; j < TT; ++j)
#pragma unroll
    for (int c = 0; c < NB; ++c) acc[j][c] = v16i{};

  v4i cur[TT][4], wst[WT];
#pragma unroll
  for (int j = 0; j < TT; ++j) load_step<ALIGNED>(cur[j], rs, base, off[j], nrec);
#pragma unroll
  for (int k = 0; k < WT; ++k) wflat0[tid + 64 * NW * k] = wsrc(0, tid + 64 * NW * k);
  __syncthreads();
  for (int s = 0; s < a.S; ++s) {
    v4i nxt[TT][4];
    const bool more = s + 1 < a.S;  // uniform
    const int b = s & 1;
    if (more) {
#pragma unroll
      for (int j = 0; j < TT; ++j) load_step<ALIGNED>(nxt[j], rs, base, off[j] + 128 * (s + 1), nrec);
#pragma unroll
      for (int k = 0; k < WT; ++k) wst[k] = wsrc(s + 1, tid + 64 * NW * k);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      v4i W[NB];
#pragma unroll
      for (int c = 0; c < NB; ++c) W[c] = wl[b][q][c][lane];
#pragma unroll
      for (int j = 0; j < TT; ++j) {
        const v4i A = a_operand(cur[j], q);
#pragma unroll
        for (int c = 0; c < NB; ++c)
          acc[j][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, W[c], acc[j][c], 0, 0, 0);
      }
    }
    if (more) {
      // the other buffer was last read in step s - 1, before the last barrier
      v4i* const wnext = b ? wflat0 : wflat1;
#pragma unroll
      for (int k = 0; k < WT; ++k) wnext[tid + 64 * NW * k] = wst[k];
#pragma unroll
      for (int j = 0; j < TT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) cur[j][i] = nxt[j][i];
    }
    __syncthreads();
  }

  // Y: lane holds column r of each tile and rows 8 (v >> 2) + 4 h + (v & 3)
  const int ncomp = 2 * a.B;
  const long long out_row = (long long)a.F * ncomp;
  int corr[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) corr[c] = a.corr[((long long)f * a.NBT + a.c0 + c) * 32 + r];
  int32_t* const out = a.beams + (long long)f * ncomp + 32 * a.c0 + r;
  auto write = [&](auto past_caches) {
#pragma unroll
    for (int j = 0; j < TT; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int t = tbase + 32 * j + 8 * (v >> 2) + 4 * h + (v & 3);
        if (t < a.T) {
#pragma unroll
          for (int c = 0; c < NB; ++c)
            if (32 * (a.c0 + c) + r < ncomp) {
              int32_t* const o = out + (long long)t * out_row + 32 * c;
              if constexpr (decltype(past_caches)::value)
                __builtin_nontemporal_store(acc[j][c][v] - corr[c], o);
              else
                *o = acc[j][c][v] - corr[c];
            }
        }
      }
  };
  // Past the caches if rows are whole 64-byte sectors, microseconds through / past
  // them: N = 96, F = 8, T = 174762, B = 48 191 / 118; N = 2048, F = 8, T = 8192,
  // B = 64 47.2 / 45.5.  Other rows share sectors with the next channel's, which
  // L2 has to join: N = 96, F = 8, T = 174762, B = 1 62 / 71; N = 224, F = 8, T =
  // 1170, B = 1 10.8 / 12.0; N = 2048, F = 16, T = 32768, B = 3 224 / 237, B = 50
  // 332 / 364; N = 1728, F = 3, T = 40000, B = 45 57 / 66.  (A few gain all the
  // same, N = 1264, F = 5, T = 35072, B = 45 91 / 79, by no rule in sight.)
  if (a.B % 8 == 0)
    write(std::true_type{});
  else
    write(std::false_type{});
}

template <int NB, int TT, int NW, bool ALIGNED>
hipError_t launch_nb(BeamArgs a, hipStream_t stream) {
  const int rows = NW * TT * 32;
  a.tblocks = (a.T + rows - 1) / rows;
  const long long grid = (long long)a.F * a.tblocks;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((beam_kernel<NB, TT, NW, ALIGNED>), dim3((unsigned)grid), dim3(64 * NW), 0,
                     stream, a);
  return hipGetLastError();
}

// Time tiles and waves: registers hold TT x NB accumulators and two steps of
// samples.  Three or four tiles take 512 rows per workgroup (one a CU) if the
// last round of workgroups leaves few CUs idle and there are several steps (N =
// 2048, F = 16, T = 32768, B = 64, four rounds: 366 us against 468 with 128 rows;
// but N = 1264, F = 5, T = 35072, B = 45, 345 workgroups: 120 against 111; N =
// 864, F = 3, T = 20864, B = 48, 123 workgroups: 31 against 24; and N = 64, F =
// 64, T = 16384, B = 40, whose time is the output's: 109 against 93).  Unaligned rows with one or two tiles take one
// time tile (N = 1090, F = 8, T = 20011, B = 20: 81 against 101 with two).
template <int NB, bool ALIGNED>
hipError_t launch_rows(const BeamArgs& a, hipStream_t stream) {
  if constexpr (NB > 4) {
    return launch_nb<NB, 1, 8, ALIGNED>(a, stream);
  } else if constexpr (NB > 2) {
    const long long grid = (long long)a.F * ((a.T + 511) / 512);
    if (a.S > 1 && (grid + a.cus - 1) / a.cus * a.cus * 5 <= grid * 6)
      return launch_nb<NB, 2, 8, ALIGNED>(a, stream);
    return launch_nb<NB, 1, 4, ALIGNED>(a, stream);
  } else {
    return launch_nb<NB, ALIGNED ? 2 : 1, 4, ALIGNED>(a, stream);
  }
}

template <int NB>
hipError_t launch_aligned_or_not(const BeamArgs& a, bool aligned, hipStream_t stream) {
  return aligned ? launch_rows<NB, true>(a, stream) : launch_rows<NB, false>(a, stream);
}

}  // namespace

hipError_t launch_beams(BeamArgs a, int nb, bool aligned, hipStream_t stream) {
  // a launch reads the weight operands and offset terms of component tiles
  // c0 .. c0 + nb - 1, which must lie inside the NBT tiles the plan holds
  if (nb < 1 || nb > kBeamTiles || a.c0 < 0 || a.c0 + nb > a.NBT) return hipErrorInvalidValue;
  switch (nb) {
    case 1: return launch_aligned_or_not<1>(a, aligned, stream);
    case 2: return launch_aligned_or_not<2>(a, aligned, stream);
    case 3: return launch_aligned_or_not<3>(a, aligned, stream);
    case 4: return launch_aligned_or_not<4>(a, aligned, stream);
    case 5: return launch_aligned_or_not<5>(a, aligned, stream);
    case 6: return launch_aligned_or_not<6>(a, aligned, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace xeng
