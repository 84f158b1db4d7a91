// The kernel of small arrays (at most 128 inputs): one workgroup of four waves
// correlates 128 / P whole channels over a time slice, P = 16, 32, 64 or 128
// columns per channel (Sec. IV-C, "Full Correlation").
//
// On 128 x 128 tiles a channel of 64 inputs leaves three quarters of the
// matrix work and half of every staged row unused, and short frames wait for
// their loads chunk by chunk at two workgroups a CU.  Here a stage of 64
// samples x 128 columns holds as many channels as fit, each at a multiple of P,
// and only the blocks inside a channel are multiplied.
//
// Blocks of 32 x 32, four column fragments: P = 128 has six off the diagonal
// and four on it, P = 64 one and two a channel, P = 32 one on the diagonal,
// P = 16 half of one.  An off-diagonal block takes two accumulators, a
// diagonal one a single D = Re + Im + 15 Sr_i (see xcorr_chan.hip), so every
// wave issues 4, 2 or 1 MFMAs a k-step:
//   P = 128  waves 0..2 two off-diagonal blocks each, wave 3 the diagonal ones
//   P = 64   waves 0, 2 the off-diagonal block of channel 0, 1; waves 1, 3
//            its two diagonal ones
//   P <= 32  wave w the diagonal block of fragment w
//
// P <= 64: what bounds a short frame is the chain load -> stage -> fragments ->
// MFMA of each chunk, so the waves share nothing: wave w takes every fourth
// chunk of the slice, all blocks of it, through a stage of its own without a
// barrier, and the four waves' sums meet once at the end.  P = 128 has too many
// accumulators for that: the four waves share a stage, double-buffered.
//
// With several slices, each stores its own partial triangles and
// chan_reduce_kernel sums them into vis.
//
// Measured, whole call, microseconds, 128 x 128 tiles -> here:
//   N = 16,  F = 1,   T = 256     8.0 ->  5.2   two launches and events -> one launch
//   N = 64,  F = 4,   T = 8192   21.2 -> 11.9   launches and the reduction's latency
//   N = 96,  F = 64,  T = 8192   51.6 -> 31.8
//   N = 128, F = 256, T = 8192  117.9 -> 86.8   3.1 TB/s: load latency, 2 WG/CU
//   N = 128, F = 64,  T = 32768 118.5 -> 87
#include "xcorr_device.hpp"
#include "xeng_chan.hpp"

namespace xeng {

namespace {

constexpr int SM_STAGE = KC * PROW;  // one stage: 64 rows of 128 columns
constexpr int SM_SETS = 4;           // chunks of loads in flight (P = 128)
// P <= 64: code sums [128], past the exchange of accumulators (4 x 3 x 4 KiB)
// and the four waves' stages
constexpr int SM_SUMS = 4 * 3 * 4096;
static_assert(4 * SM_STAGE <= SM_SUMS, "the waves' stages lie below the sums");
static_assert(4 * 32 * 33 * 4 <= 2 * SM_STAGE, "the transposes fit the stages");

// A wave's blocks: off-diagonal (oi[k], oj[k]), k < NO, and diagonal dg[k], k < ND.
template <int P, int W>
struct SmallRole;
template <int W>
struct SmallRole<128, W> {
  static constexpr int NO = W < 3 ? 2 : 0, ND = W < 3 ? 0 : 4;
  static constexpr int oi[2] = {0, W == 0 ? 2 : 1};
  static constexpr int oj[2] = {W + 1, W == 0 ? 3 : W == 1 ? 3 : 2};
  static constexpr int dg[4] = {0, 1, 2, 3};
};
template <int W>
struct SmallRole<64, W> {
  static constexpr int NO = W & 1 ? 0 : 1, ND = W & 1 ? 2 : 0;
  static constexpr int oi[2] = {W & 2, 0}, oj[2] = {(W & 2) + 1, 0};
  static constexpr int dg[4] = {W & 2, (W & 2) + 1, 0, 0};
};
template <int W>
struct SmallRole<32, W> {
  static constexpr int NO = 0, ND = 1;
  static constexpr int oi[2] = {0, 0}, oj[2] = {0, 0};
  static constexpr int dg[4] = {W, 0, 0, 0};
};
template <int W>
struct SmallRole<16, W> : SmallRole<32, W> {};

// Row of register v in a lane's share of a 32 x 32 MFMA block.
__device__ __forceinline__ int small_row(int v, int lane) {
  return (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
}

// Write the blocks of wave W's role (products of codes over T samples): S holds
// the code sums of the 128 columns, mt a 32 x 33 matrix of this wave's.
template <int P, int W>
__device__ __forceinline__ void small_write(const ChanArgs& a, int f0, int slice, int T,
                                            const v16i* re, const v16i* im, const v16i* dd,
                                            const int2* S, int* mt, int lane) {
  typedef SmallRole<P, W> R;
  const int N = a.N;
  const long long NB = (long long)N * (N + 1) / 2;
  int32_t* out = a.partial ? a.partial + 2 * NB * ((long long)slice * a.F) : a.vis;
  const int T128 = 128 * T;
  const int lj = lane & 31;
  // baseline (i, j) of channel f0 + k from its codes' products
  auto put = [&](int k, int i, int j, int xre, int xim, int2 si, int2 sj) {
    if (f0 + k >= a.F || i > j || j >= N) return;
    int32_t* q = out + 2 * ((long long)(f0 + k) * NB + pair_index(i, j, N));
    int2 v = make_int2(xre + T128 - 8 * (si.x + si.y + sj.x + sj.y),
                       i == j ? 0 : xim - 8 * (si.y - si.x) + 8 * (sj.y - sj.x));
    if (a.write_mode == WM_ADD) {
      const int2 o = *reinterpret_cast<const int2*>(q);
      v.x += o.x;
      v.y += o.y;
    }
    *reinterpret_cast<int2*>(q) = v;
  };
#pragma unroll
  for (int k = 0; k < R::NO; ++k) {
    const int ci = 32 * R::oi[k], cj = 32 * R::oj[k];
    const int2 sj = S[cj + lj];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int di = small_row(v, lane);
      const int2 si = S[ci + di];
      put(ci / P, ci % P + di, cj % P + lj, re[k][v], im[k][v] - 15 * si.x, si, sj);
    }
  }
#pragma unroll
  for (int k = 0; k < R::ND; ++k) {
    // the block's transpose through LDS (this wave's; its LDS operations
    // complete in order)
    const int c0 = 32 * R::dg[k];
#pragma unroll
    for (int v = 0; v < 16; ++v) mt[small_row(v, lane) * 33 + lj] = dd[k][v];
    const int2 sj = S[c0 + lj];
    const int j = c0 + lj;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int di = small_row(v, lane), i = c0 + di;
      const int x = dd[k][v], t = mt[lj * 33 + di];
      const int2 si = S[i];
      if (P == 16 && i / P != j / P) continue;  // the block's two channels do not mix
      put(j / P, i % P, j % P, (x + t - 15 * (si.x + sj.x)) >> 1, (x - t - 15 * (si.x - sj.x)) >> 1,
          si, sj);
    }
  }
}

// The whole work of wave W, P = 128: the waves share every chunk.
template <int P, int W, bool FAST>
__device__ __forceinline__ void small_shared(const ChanArgs& a, int f0, int slice, int t_begin,
                                           int t_end, uint8_t* lds) {
  typedef SmallRole<P, W> R;
  constexpr int CH = BT / P;  // channels of the workgroup
  const int tid = threadIdx.x, lane = tid & 63;
  const int N = a.N;
  // staging: two 16-byte pieces, rows `row` and row + 32 of column segment seg
  // (rows in the order that keeps LDS writes free of conflicts; see StageRole)
  const int seg = tid & 7, rq = tid >> 3;
  const int row = 4 * (rq & 1) + ((rq >> 1) & 3) + 8 * (rq >> 3);
  const int ck = 16 * seg / P, n0 = 16 * seg % P;  // the segment's channel and first input
  const bool there = f0 + ck < a.F && n0 < N;
  // fast loads of absent pieces read channel f0, input 0 instead (never written)
  const int col = there ? ck * N + n0 : 0;
  const uint32_t off = (uint32_t)row * (uint32_t)a.row_stride + (uint32_t)col;
  const int s32 = (int)(32 * a.row_stride);
  const int len = t_end - t_begin, nchunks = (len + KC - 1) / KC;
  const int t_fast = fast_rows(a.t_frame, N, min(f0 + CH, a.F) - 1, a.F);
  const int len_fast = FAST ? min(t_end, t_fast) - t_begin : 0;
  const int nfast = len_fast > 0 ? len_fast / KC : 0;
  const uint8_t* rows = a.samples + (long long)t_begin * a.row_stride + (long long)f0 * N;
  auto load = [&](v4i (&raw)[2], int c) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(rows + (long long)c * KC * a.row_stride), (short)0, 0x7fffffff, 0x00020000);
    raw[0] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
    raw[1] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, s32, 0));
  };
  auto load_edge = [&](v4i (&raw)[2], int c) {
    const int z = (int)0x88888888u, t = t_begin + c * KC + row;
    raw[0] = raw[1] = v4i{z, z, z, z};
    if (!there) return;
    raw[0] = load_piece_edge(a.samples, a.row_stride, f0 + ck, N, n0, t, t_end, t_fast);
    raw[1] = load_piece_edge(a.samples, a.row_stride, f0 + ck, N, n0, t + 32, t_end, t_fast);
  };
  auto stage = [&](const v4i (&raw)[2], int c) {
    uint8_t* d = lds + (c & 1) * SM_STAGE + row * PROW + 16 * seg;
    *reinterpret_cast<v4i*>(d) = raw[0];
    *reinterpret_cast<v4i*>(d + 32 * PROW) = raw[1];
  };

  v16i re[2] = {v16i{}, v16i{}}, im[2] = {v16i{}, v16i{}}, dd[4] = {v16i{}, v16i{}, v16i{}, v16i{}};
  uint32_t sr = 0u, sm = 0u;
  const int lane_rd = lane_read_offset<FORM_I8>(lane);
  auto compute = [&](int c) {
    const uint8_t* p = lds + (c & 1) * SM_STAGE + lane_rd;
    constexpr int c15 = 0x0F0F0F0F;
    v2i w[KC / 16][4];  // the chunk's transposed reads, all at once
#pragma unroll
    for (int s = 0; s < KC / 16; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) w[s][q] = lds_tr8(p + 16 * s * PROW + 32 * q);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t br = 0u, bm = 0u;  // bytewise within the chunk (eight codes a byte)
#pragma unroll
    for (int s = 0; s < KC / 16; ++s) {
      v2i r[4], m[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        r[q] = hi_codes(w[s][q]);
        m[q] = lo_codes(w[s][q]);
      }
      br = badd(r[W].x, r[W].y, br);
      bm = badd(m[W].x, m[W].y, bm);
#pragma unroll
      for (int k = 0; k < R::NO; ++k) {
        const int i = R::oi[k], j = R::oj[k];
        const v4i A = v4i{m[i].x, m[i].y, r[i].x, r[i].y};
        const v4i B = v4i{m[j].x, m[j].y, r[j].x, r[j].y};
        const v4i Y = v4i{r[j].x, r[j].y, m[j].x ^ c15, m[j].y ^ c15};
        re[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, B, re[k], 0, 0, 0);
        im[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, Y, im[k], 0, 0, 0);
      }
#pragma unroll
      for (int k = 0; k < R::ND; ++k) {
        const int i = R::dg[k];
        const v4i A = v4i{m[i].x, m[i].y, r[i].x, r[i].y};
        const v4i Z = v4i{m[i].x + r[i].x, m[i].y + r[i].y, r[i].x + (m[i].x ^ c15),
                          r[i].y + (m[i].y ^ c15)};
        dd[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, Z, dd[k], 0, 0, 0);
      }
    }
    sr = __builtin_amdgcn_udot4(br, 0x01010101u, sr, false);
    sm = __builtin_amdgcn_udot4(bm, 0x01010101u, sm, false);
  };

  // Whole chunks inside the frame, in groups of four, with loads four chunks
  // ahead (past the last one they read it again) and one barrier a chunk: a
  // wave stages chunk c into the buffer of chunk c - 2, which every wave left
  // before the barrier of chunk c - 1.
  const int nsteady = nfast / SM_SETS * SM_SETS;
  if (nsteady > 0) {
    v4i raw[SM_SETS][2];
#pragma unroll
    for (int u = 0; u < SM_SETS; ++u) {
      load(raw[u], u);
      // in the loop's order, so that its waits (loads return in order) are for
      // the oldest set alone
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int c = 0; c < nsteady; c += SM_SETS) {
#pragma unroll
      for (int u = 0; u < SM_SETS; ++u) {
        stage(raw[u], c + u);
        load(raw[u], min(c + u + SM_SETS, nfast - 1));
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        compute(c + u);
      }
    }
  }
  // the rest, one chunk ahead
  v4i cur[2];
  auto load_one = [&](int c) {
    if (c < nfast) load(cur, c);
    else load_edge(cur, c);
  };
  if (nsteady < nchunks) load_one(nsteady);
  for (int c = nsteady; c < nchunks; ++c) {
    stage(cur, c);
    if (c + 1 < nchunks) load_one(c + 1);
    __syncthreads();
    compute(c);
  }

  // code sums: lanes l and l + 32 hold the two halves of every k-step
  int2* S = reinterpret_cast<int2*>(lds + 2 * SM_STAGE);
  sr += __shfl_xor(sr, 32);
  sm += __shfl_xor(sm, 32);
  if (lane < 32) S[32 * W + lane] = make_int2((int)sr, (int)sm);
  __syncthreads();  // the sums are complete, and the stages free

  small_write<P, W>(a, f0, slice, nchunks * KC, re, im, dd, S,
                    reinterpret_cast<int*>(lds) + W * 32 * 33, lane);
}

// P <= 64: every wave takes every fourth chunk for itself, all four fragments,
// through its own 10 KiB of LDS with no barrier (a wave's LDS operations
// complete in order), and the four waves' accumulators are added at the end.  A
// chunk's chain of dependent steps is then paid once per four chunks, and a
// wave's independent accumulators (4, or 8 at P = 64) keep the matrix cores
// busy meanwhile.
template <int P, bool FAST>
__device__ __forceinline__ void small_private(const ChanArgs& a, int f0, int slice, int t_begin,
                                              int t_end, int wave, uint8_t* lds) {
  constexpr int CH = BT / P, NOFF = P == 64 ? 2 : 0;
  const int lane = threadIdx.x & 63;
  const int N = a.N;
  // staging: eight 16-byte pieces a lane, rows row0 + 8 k of column segment seg
  const int seg = lane & 7, row0 = lane >> 3;
  const int ck = 16 * seg / P, n0 = 16 * seg % P;  // the segment's channel and first input
  const bool there = f0 + ck < a.F && n0 < N;
  // fast loads of absent pieces read channel f0, input 0 instead (never written)
  const uint32_t off = (uint32_t)row0 * (uint32_t)a.row_stride + (uint32_t)(there ? ck * N + n0 : 0);
  const int s8 = (int)(8 * a.row_stride);
  const int len = t_end - t_begin, nchunks = (len + KC - 1) / KC;
  const int t_fast = fast_rows(a.t_frame, N, min(f0 + CH, a.F) - 1, a.F);
  const int len_fast = FAST ? min(t_end, t_fast) - t_begin : 0;
  const int nfast = len_fast > 0 ? len_fast / KC : 0;
  const uint8_t* rows = a.samples + (long long)t_begin * a.row_stride + (long long)f0 * N;
  uint8_t* const my = lds + wave * SM_STAGE;
  auto load = [&](v4i (&raw)[8], int c) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(rows + (long long)c * KC * a.row_stride), (short)0, 0x7fffffff, 0x00020000);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      raw[k] = __builtin_bit_cast(v4i,
                                  __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, k * s8, 0));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_edge = [&](v4i (&raw)[8], int c) {
    const int z = (int)0x88888888u;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      raw[k] = there ? load_piece_edge(a.samples, a.row_stride, f0 + ck, N, n0,
                                       t_begin + c * KC + row0 + 8 * k, t_end, t_fast)
                     : v4i{z, z, z, z};
  };
  auto stage = [&](const v4i (&raw)[8]) {
#pragma unroll
    for (int k = 0; k < 8; ++k)
      *reinterpret_cast<v4i*>(my + (row0 + 8 * k) * PROW + 16 * seg) = raw[k];
  };
  v16i re[2] = {v16i{}, v16i{}}, im[2] = {v16i{}, v16i{}}, dd[4] = {v16i{}, v16i{}, v16i{}, v16i{}};
  uint32_t sr[4] = {0u, 0u, 0u, 0u}, sm[4] = {0u, 0u, 0u, 0u};
  const uint8_t* const rd = my + lane_read_offset<FORM_I8>(lane);
  constexpr int c15 = 0x0F0F0F0F;
  auto compute = [&]() {
    // all of the chunk's transposed reads go out first: the chain from a read
    // to its product is paid once a chunk, not once a k-step
    v2i w[KC / 16][4];
#pragma unroll
    for (int s = 0; s < KC / 16; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) w[s][q] = lds_tr8(rd + 16 * s * PROW + 32 * q);
    __builtin_amdgcn_sched_barrier(0);
    // code sums bytewise within the chunk (eight codes of at most 15 a byte)
    uint32_t br[4] = {0u, 0u, 0u, 0u}, bm[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int s = 0; s < KC / 16; ++s) {
      v2i r[4], m[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        r[q] = hi_codes(w[s][q]);
        m[q] = lo_codes(w[s][q]);
        br[q] = badd(r[q].x, r[q].y, br[q]);
        bm[q] = badd(m[q].x, m[q].y, bm[q]);
        const v4i A = v4i{m[q].x, m[q].y, r[q].x, r[q].y};
        const v4i Z = v4i{m[q].x + r[q].x, m[q].y + r[q].y, r[q].x + (m[q].x ^ c15),
                          r[q].y + (m[q].y ^ c15)};
        dd[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, Z, dd[q], 0, 0, 0);
      }
#pragma unroll
      for (int k = 0; k < NOFF; ++k) {
        const int i = 2 * k, j = 2 * k + 1;
        const v4i A = v4i{m[i].x, m[i].y, r[i].x, r[i].y};
        const v4i B = v4i{m[j].x, m[j].y, r[j].x, r[j].y};
        const v4i Y = v4i{r[j].x, r[j].y, m[j].x ^ c15, m[j].y ^ c15};
        re[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, B, re[k], 0, 0, 0);
        im[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A, Y, im[k], 0, 0, 0);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sr[q] = __builtin_amdgcn_udot4(br[q], 0x01010101u, sr[q], false);
      sm[q] = __builtin_amdgcn_udot4(bm[q], 0x01010101u, sm[q], false);
    }
  };
  // whole chunks inside the frame: wave, wave + 4, ..., the next one's loads
  // behind each (past the last one they read it again; two in flight gained
  // nothing)
  const int nw = (nfast - wave + 3) >> 2, last = wave + 4 * (nw - 1);
  if (nw > 0) {
    v4i raw[8];
    load(raw, wave);
    for (int k = 0; k < nw; ++k) {
      stage(raw);
      load(raw, min(wave + 4 * k + 4, last));
      compute();
    }
  }
  // the frame's last row and a ragged chunk
  for (int c = max(nfast, 0); c < nchunks; ++c) {
    if ((c & 3) != wave) continue;  // uniform
    v4i r[8];
    load_edge(r, c);
    stage(r);
    compute();
  }

  // The waves' sums: code sums by LDS atomics; accumulators in rounds of one a
  // wave, which the wave that writes it collects from the other three.
  int* Sw = reinterpret_cast<int*>(lds + SM_SUMS);
  __syncthreads();  // the stages are free
  Sw[threadIdx.x] = 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int x = (int)(sr[q] + __shfl_xor(sr[q], 32)), y = (int)(sm[q] + __shfl_xor(sm[q], 32));
    if (lane < 32) {
      atomicAdd(&Sw[2 * (32 * q + lane)], x);
      atomicAdd(&Sw[2 * (32 * q + lane) + 1], y);
    }
  }
  int* const box = reinterpret_cast<int*>(lds);  // [dest wave][3][16][64]
  auto give = [&](int dest, const v16i& x) {
    if (dest == wave) return;  // uniform
    int* d = box + (dest * 3 + ((wave - dest - 1) & 3)) * 1024 + lane;
#pragma unroll
    for (int v = 0; v < 16; ++v) d[64 * v] = x[v];
  };
  auto take = [&](v16i& x) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] += box[(wave * 3 + k) * 1024 + 64 * v + lane];
  };
  const int2* S = reinterpret_cast<const int2*>(Sw);
  int* mt = reinterpret_cast<int*>(lds) + wave * 32 * 33;
  const int T = nchunks * KC;
  if constexpr (P == 64) {
    // wave 2 c: channel c's off-diagonal block; wave 2 c + 1: its diagonal ones
    v16i x[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      give(0, k ? im[0] : re[0]);
      give(1, dd[k]);
      give(2, k ? im[1] : re[1]);
      give(3, dd[2 + k]);
      x[k] = wave == 0 ? (k ? im[0] : re[0])
                       : wave == 1 ? dd[k] : wave == 2 ? (k ? im[1] : re[1]) : dd[2 + k];
      __syncthreads();
      take(x[k]);
      __syncthreads();
    }
    switch (wave) {
      case 0: small_write<P, 0>(a, f0, slice, T, &x[0], &x[1], nullptr, S, mt, lane); break;
      case 1: small_write<P, 1>(a, f0, slice, T, nullptr, nullptr, x, S, mt, lane); break;
      case 2: small_write<P, 2>(a, f0, slice, T, &x[0], &x[1], nullptr, S, mt, lane); break;
      default: small_write<P, 3>(a, f0, slice, T, nullptr, nullptr, x, S, mt, lane); break;
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) give(q, dd[q]);
    v16i x = wave == 0 ? dd[0] : wave == 1 ? dd[1] : wave == 2 ? dd[2] : dd[3];
    __syncthreads();
    take(x);
    __syncthreads();
    switch (wave) {
      case 0: small_write<P, 0>(a, f0, slice, T, nullptr, nullptr, &x, S, mt, lane); break;
      case 1: small_write<P, 1>(a, f0, slice, T, nullptr, nullptr, &x, S, mt, lane); break;
      case 2: small_write<P, 2>(a, f0, slice, T, nullptr, nullptr, &x, S, mt, lane); break;
      default: small_write<P, 3>(a, f0, slice, T, nullptr, nullptr, &x, S, mt, lane); break;
    }
  }
}

}  // namespace

template <int P, bool FAST>
__global__ void __launch_bounds__(256, P < 64 ? 3 : 2) xcorr_small_kernel(ChanArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[(P == 128 ? 2 * SM_STAGE : SM_SUMS) + BT * 8];
  const int b = blockIdx.x;
  const int s = b % a.nslices, f0 = b / a.nslices * (BT / P);
  const int t_begin = a.t0 + s * a.slice_len;
  const int t_end = min(a.t1, t_begin + a.slice_len);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);  // uniform
  if constexpr (P == 128) {
    // the diagonal role has the most vector work: roles rotate over the
    // workgroups of a CU, whose waves w share SIMD w
    switch ((wave + b) & 3) {
      case 0: small_shared<P, 0, FAST>(a, f0, s, t_begin, t_end, lds); break;
      case 1: small_shared<P, 1, FAST>(a, f0, s, t_begin, t_end, lds); break;
      case 2: small_shared<P, 2, FAST>(a, f0, s, t_begin, t_end, lds); break;
      default: small_shared<P, 3, FAST>(a, f0, s, t_begin, t_end, lds); break;
    }
  } else {
    small_private<P, FAST>(a, f0, s, t_begin, t_end, wave, lds);
  }
}

int small_columns(int N) { return N <= 16 ? 16 : N <= 32 ? 32 : N <= 64 ? 64 : 128; }

hipError_t launch_small(const ChanArgs& a, bool fast, hipStream_t stream) {
  if (a.N < 1 || a.N > BT || a.nslices < 1 || a.slice_len < 1 || a.slice_len % KC != 0 ||
      (long long)(a.nslices - 1) * a.slice_len >= a.t1 - a.t0)
    return hipErrorInvalidValue;  // every slice holds samples
  const int P = small_columns(a.N), ch = BT / P;
  const long long grid = (long long)((a.F + ch - 1) / ch) * a.nslices;
  if (grid <= 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 g((unsigned)grid), b(256);
#define XENG_SMALL(PP)                                                                       \
  do {                                                                                       \
    if (fast) hipLaunchKernelGGL((xcorr_small_kernel<PP, true>), g, b, 0, stream, a);        \
    else hipLaunchKernelGGL((xcorr_small_kernel<PP, false>), g, b, 0, stream, a);            \
  } while (0)
  switch (P) {
    case 16: XENG_SMALL(16); break;
    case 32: XENG_SMALL(32); break;
    case 64: XENG_SMALL(64); break;
    default: XENG_SMALL(128); break;
  }
#undef XENG_SMALL
  return hipGetLastError();
}

}  // namespace xeng
