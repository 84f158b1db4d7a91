// The packed path's correlation kernel: 256 x 128 baselines per workgroup on
// FP6 MFMA, operands as xeng_pack.hip laid them out (xeng_packed.hpp).
//
// A 4-bit code is an FP6 e2m3 number as it stands, and the FP6 matrix cores
// run twice the rate of the int8 and FP8 ones: MFMA-only code reaches 7.35 to
// 7.55 POP/s on codes (1.85 GHz, at the power limit; mfma_ceiling.hip) against
// 3.53 to 3.64 in int8 and 4.93 in FP8.  The sums of products of codes are integers below 450 T < 2^24 over
// one segment (T <= XENG_F8_FLUSH_MAX), exact in f32 in any order.
//
// What bounds it is power: on 2048 inputs, 16 channels, 32768 samples it takes
// 1.80 ms (packing excluded; 3.17 ms for the int8 tiles), the MFMA pipe busy
// 66% of the cycles at 1.79 GHz.  With all loads and LDS reads taken out (a
// timing copy) it takes 1.38 ms at 1.71 GHz, so what costs most beside the
// MFMAs is moving operands: hence tiles as large as 512 registers a lane
// allow, whose four waves are alone on their SIMDs.
#include "xcorr_device.hpp"
#include "xeng_packed.hpp"

namespace xeng {

namespace {

constexpr int PK_STAGE = 4 * 8 * FRAG_BYTES;     // one LDS stage: 4 steps x 8 fragments
constexpr int PK_MAT = 32 * 33;                  // a diagonal block in LDS (one pad column)

// An FP6 operand: [r(16), m(16)], six words (the MFMA takes eight and ignores
// the last two).
__device__ __forceinline__ v8i op6(v4i lo, v2i hi) {
  return v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, 0, 0};
}

// Words w and w + 3 of a rotated operand from [r, m] (the sign of a 6-bit code
// is its top bit): rows take [m, -r], columns [-m, r], so that with either
// one rotated the product is Im = sum m_i r_j - r_i m_j.  The copy is made
// here: the compiler would otherwise make it where the operand is loaded, and
// wait for the load there.
template <bool COL>
__device__ __forceinline__ void rot6(v8i& o, const v8i& x, int w) {
  const uint32_t sign[3] = {0x20820820u, 0x08208208u, 0x82082082u};
  // word w of the sixteen imaginary (real) codes sits in word 3 + w (w)
  if (!COL) {
    int m = x[3 + w];
    asm volatile("" : "+v"(m));
    o[w] = m;
    o[3 + w] = (int)((uint32_t)x[w] ^ sign[w]);
  } else {
    int r = x[w];
    asm volatile("" : "+v"(r));
    o[3 + w] = r;
    o[w] = (int)((uint32_t)x[3 + w] ^ sign[w]);
  }
}

__device__ __forceinline__ v4i ld16(__amdgpu_buffer_rsrc_t rs, int v, int s) {
  return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, v, s, 0));
}
__device__ __forceinline__ v2i ld8(__amdgpu_buffer_rsrc_t rs, int v, int s) {
  return __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(rs, v, s, 0));
}

// Scalar resource of an operand stream; a segment's steps of one channel stay
// below 2^31 bytes (32768 samples of 32768 inputs take 1.6e9).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t stream_rsrc(const uint8_t* q) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)q, (short)0, 0x7fffffff, 0x00020000);
}

__device__ __forceinline__ v16f mfma6(const v8i& a, const v8i& b, const v16f& c) {
  // format 2 = FP6 e2m3 for both operands; no scales: the sums are exact
  // multiples of 1 / 64 (see f6_int)
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 2, 0, 0, 0, 0);
}

// A sum of products of codes: a code u reads u / 8, so the sum is an integer
// below 2^24 over 64 (exact in f32).
__device__ __forceinline__ int f6_int(float x) { return (int)(x * 64.0f); }

__device__ __forceinline__ v4i lds16(const uint8_t* p) { return *reinterpret_cast<const v4i*>(p); }
__device__ __forceinline__ v2i lds8(const uint8_t* p) { return *reinterpret_cast<const v2i*>(p); }

// Tile p of a channel -> (I, J): macro row I (inputs 256 I..), and either its
// diagonal (J < 0: the triangle of those 256 inputs) or 128-column block J.
__device__ __forceinline__ void packed_tile_of(int p, int blocks, int& I, int& J) {
  int i = 0;
  for (;;) {
    const int n = 1 + max(0, blocks - 2 * i - 2);
    if (p < n) break;
    p -= n;
    ++i;
  }
  I = i;
  J = p == 0 ? -1 : 2 * i + 1 + p;
}

// Offset corrections of one input (see row_corr): with its code sums over the
// T samples, Re V_ij += p_i + p_j + 128 T and Im V_ij += q_i - q_j.
__device__ __forceinline__ int2 pq_corr(int sr, int sm) {
  return make_int2(-8 * (sr + sm), 8 * (sr - sm));
}

// Where a tile's results go.
struct TileOut {
  int32_t* base;  // the channel's packed triangle
  int2* part;     // this item's partial blocks, or NULL
  int N, T, mode;
};

// Sixteen baselines of a lane: rows i0 + blk_row(v), column j of block `blk`.
__device__ __forceinline__ int blk_row16(int v, int lane) {
  return (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
}

__device__ __forceinline__ void put16(const TileOut& o, int blk, int i0, int j0, int lane,
                                      const int (&vr)[16], const int (&vi)[16]) {
  if (o.part) {
    int2* d = o.part + (long long)blk * 1024 + lane;
#pragma unroll
    for (int v = 0; v < 16; ++v) d[64 * v] = make_int2(vr[v], vi[v]);
    return;
  }
  const int j = j0 + (lane & 31);
  if (o.mode == WM_ADD) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // eight at a time: fewer live registers
      int b[8], r[8], m[8];
      uint32_t ok = 0u;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + blk_row16(8 * h + u, lane);
        ok |= (uint32_t)(i < o.N && j < o.N && j >= i) << u;
        b[u] = pair_index(i, j, o.N);
        r[u] = vr[8 * h + u];
        m[u] = i == j ? 0 : vi[8 * h + u];
      }
      add_pairs(o.base, b, r, m, ok);
    }
    return;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = i0 + blk_row16(v, lane);
    if (i < o.N && j < o.N && j >= i)
      *reinterpret_cast<int2*>(o.base + 2 * pair_index(i, j, o.N)) =
          make_int2(vr[v], i == j ? 0 : vi[v]);
  }
}

// An off-diagonal block from its two accumulators; ci / cj: corrections of its
// first row and column (LDS).
__device__ __forceinline__ void put_off(const TileOut& o, int blk, int i0, int j0, const v16f& re,
                                        const v16f& im, const int2* ci, const int2* cj, int lane) {
  if (i0 >= o.N || j0 >= o.N) return;
  const int2 b = cj[lane & 31];
  int vr[16], vi[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int2 a = ci[blk_row16(v, lane)];
    vr[v] = f6_int(re[v]) + a.x + b.x + 128 * o.T;
    vi[v] = f6_int(im[v]) + a.y - b.y;
  }
  put16(o, blk, i0, j0, lane, vr, vi);
}

// A diagonal block from its one accumulator D = Re + Im: Re is symmetric and
// Im antisymmetric, so Re = (D + D^T) / 2 and Im = (D - D^T) / 2, exactly.
// The transpose comes through `m` (LDS, 32 x 33, this wave's; a wave's LDS
// operations complete in order).
__device__ __forceinline__ void put_diag(const TileOut& o, int blk, int i0, const v16f& d,
                                         const int2* c, int* m, int lane) {
  if (i0 >= o.N) return;
  const int lj = lane & 31;
#pragma unroll
  for (int v = 0; v < 16; ++v) m[blk_row16(v, lane) * 33 + lj] = f6_int(d[v]);
  const int2 b = c[lj];
  int vr[16], vi[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int di = blk_row16(v, lane);
    const int x = f6_int(d[v]), t = m[lj * 33 + di];
    const int2 a = c[di];
    vr[v] = ((x + t) >> 1) + a.x + b.x + 128 * o.T;
    vi[v] = di == lj ? 0 : ((x - t) >> 1) + a.y - b.y;
  }
  put16(o, blk, i0, i0, lane, vr, vi);
}

// Corrections of inputs n0 + tid (tid < cnt) from the code sums of blocks
// [sb0, sb1).
__device__ __forceinline__ void load_corr(const PackedArgs& a, int f, int n0, int cnt, int sb0,
                                          int sb1, int2* c) {
  const int tid = threadIdx.x, np = a.blocks * BT;
  if (tid >= cnt) return;
  const int2* S = a.sums + (long long)f * a.nsum * np + min(n0 + tid, np - 1);
  int sr = 0, sm = 0;
  for (int k = sb0; k < sb1; ++k) {
    const int2 v = S[(long long)k * np];
    sr += v.x;
    sm += v.y;
  }
  c[tid] = pq_corr(sr, sm);
}

// One 256 x 128 tile off the diagonal: wave w takes rows 64 w.. (two fragments)
// and all 128 columns (four), 2 x 4 blocks with a Re and an Im accumulator
// each.  The rows' operands are the wave's own and come straight from global
// memory; the columns' are staged in LDS, four steps (128 samples) at a time.
//
// A SIMD has one wave here (its accumulators alone are 256 registers), which
// issues about one instruction every four cycles and an MFMA every 32: up to
// six instructions hide behind each MFMA and a longer run of them would not.
// So everything but the MFMAs is dealt out between them, one slot per MFMA,
// with fences that keep the order: a step's MFMAs carry the LDS reads of the
// next step, the staging of the next round, and the loads of the next round
// (rows) and the one after it (columns).
__device__ __forceinline__ void off_tile(const PackedArgs& a, const TileOut& o, int f, int I,
                                         int J, int t_begin, int t_end, int wave, uint8_t* lds) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int ngrain = (t_end - t_begin) / PK_GRAIN;
  const int step_b = a.blocks * BLOCK_BYTES, round_b = 4 * step_b;
  const uint8_t* base = a.packed + ((long long)f * a.steps + t_begin / PK_STEP) * step_b;
  const __amdgpu_buffer_rsrc_t ra = stream_rsrc(base + (8 * I + 2 * wave) * FRAG_BYTES);
  const __amdgpu_buffer_rsrc_t rb = stream_rsrc(base + J * BLOCK_BYTES);
  const int va0 = 16 * lane, va1 = 1024 + 8 * lane;
  // column staging: 16-byte units e = tid + 256 k (k < 6) of a round's four
  // steps (384 units each)
  int vb[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const int e = tid + 256 * k;
    vb[k] = (e / 384) * step_b + (e % 384) * 16;
  }
  auto load_a = [&](v8i& x, int frag, int off) {  // one fragment of a step
    x = op6(ld16(ra, va0 + frag * FRAG_BYTES, off), ld8(ra, va1 + frag * FRAG_BYTES, off));
  };
  v16f re[2][4], im[2][4];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) re[x][y] = im[x][y] = v16f{};

  // One step: the real parts first, then the imaginary ones, whose rotated rows
  // the slots of the first make; the rows are free for their next load after
  // eight MFMAs.  The next step's columns are read from LDS (at `nu`) from
  // slot RD on.
  auto step = [&](auto rd, v8i (&A)[2], const v8i (&B)[4], v8i (&Bn)[4], const uint8_t* nu,
                  int oa, auto&& extra) {
    constexpr int RD = decltype(rd)::value;
    v8i R[2] = {v8i{}, v8i{}};
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int x = k & 1, q = (k & 7) >> 1;
      if (k < 8)
        re[x][q] = mfma6(A[x], B[q], re[x][q]);
      else
        im[x][q] = mfma6(R[x], B[q], im[x][q]);
      if (k >= RD && (k - RD) / 3 < 4) {
        const int n = (k - RD) / 3;
        const uint8_t* u = nu + n * FRAG_BYTES;
        if ((k - RD) % 3 == 0) Bn[n] = op6(lds16(u + 16 * lane), v2i{0, 0});
        if ((k - RD) % 3 == 1) {
          const v2i hi = lds8(u + 1024 + 8 * lane);
          Bn[n][4] = hi.x;
          Bn[n][5] = hi.y;
        }
      }
      if (k >= 1 && k < 7) rot6<false>(R[(k - 1) / 3], A[(k - 1) / 3], (k - 1) % 3);
      if (k == 8 || k == 9) load_a(A[k - 8], k - 8, oa);
      extra(k);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  constexpr int CH = 4 * 4 * FRAG_BYTES;  // a stage: 4 steps x 4 fragments
  v8i A[4][2], B0[4], B1[4];
  v4i st[6];
  auto load_b = [&](int off, int k) { st[k] = ld16(rb, vb[k], off); };
  auto stage = [&](uint8_t* d, int k) {
    *reinterpret_cast<v4i*>(d + 16 * (tid + 256 * k)) = st[k];
  };
  // the loads go out in the loop's order, so that the loop's waits (loads
  // return in order) are the same on its first round
#pragma unroll
  for (int k = 0; k < 6; ++k) load_b(0, k);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    load_a(A[s][0], 0, s * step_b);
    load_a(A[s][1], 1, s * step_b);
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) stage(lds, k);
#pragma unroll
  for (int k = 0; k < 6; ++k) load_b(ngrain > 1 ? round_b : 0, k);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 2; s < 4; ++s) {
    load_a(A[s][0], 0, s * step_b);
    load_a(A[s][1], 1, s * step_b);
  }
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q)
    B0[q] = op6(lds16(lds + q * FRAG_BYTES + 16 * lane), lds8(lds + q * FRAG_BYTES + 1024 + 8 * lane));
  __builtin_amdgcn_sched_barrier(0);
  const std::integral_constant<int, 0> at0;
  const std::integral_constant<int, 4> at4;
  for (int g = 0; g < ngrain; ++g) {
    const uint8_t* cur = lds + (g & 1) * CH;
    uint8_t* nxt = lds + ((g + 1) & 1) * CH;
    const int oa = min(g + 1, ngrain - 1) * round_b, ob = min(g + 2, ngrain - 1) * round_b;
    step(at0, A[0], B0, B1, cur + 4 * FRAG_BYTES, oa, [&](int) {});
    step(at0, A[1], B1, B0, cur + 8 * FRAG_BYTES, oa + step_b, [&](int) {});
    // stage the next round and load the one after it into the freed registers
    step(at0, A[2], B0, B1, cur + 12 * FRAG_BYTES, oa + 2 * step_b, [&](int k) {
      if (k < 12 && k % 2 == 0) stage(nxt, k / 2);
      if (k < 12 && k % 2 == 1) load_b(ob, k / 2);
    });
    // the next round is staged and this one's last step in registers once
    // every wave passes the barrier
    step(at4, A[3], B1, B0, nxt, oa + 3 * step_b, [&](int k) {
      if (k == 3) __syncthreads();
    });
  }

  __syncthreads();
  int2* ci = reinterpret_cast<int2*>(lds);
  const int sb0 = t_begin / a.sumb, sb1 = (t_end + a.sumb - 1) / a.sumb;
  load_corr(a, f, 256 * I, 256, sb0, sb1, ci);
  load_corr(a, f, 128 * J, 128, sb0, sb1, ci + 256);
  __syncthreads();
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y)
      put_off(o, (2 * wave + x) * 4 + y, 256 * I + 64 * wave + 32 * x, 128 * J + 32 * y, re[x][y],
              im[x][y], ci + 64 * wave + 32 * x, ci + 256 + 32 * y, lane);
}

// The diagonal: the triangle of 256 inputs (fragments 0..7), 28 blocks off the
// diagonal with two accumulators and 8 on it with one (both products added
// into it, see put_diag), i.e. 64 accumulators as in an off-diagonal tile, for
// 72 MFMAs a step instead of 64.  Every wave takes seven and two of them:
// wave w the fragments of its quarter 2 w, 2 w + 1 against themselves and two
// other quarters.  Local fragments: `frag`; blocks (row, column) in local
// indices; ROTC: columns rather than rows are rotated; `rot` lists them.
template <int W>
struct DiagWave;
template <>
struct DiagWave<0> {
  static constexpr int NF = 6, NR = 2;
  static constexpr bool ROTC = false;
  static constexpr int frag[6] = {0, 1, 2, 3, 4, 5};
  static constexpr int bi[7] = {0, 0, 0, 1, 1, 0, 0}, bj[7] = {1, 2, 3, 2, 3, 4, 5};
  static constexpr int dg[2] = {0, 1}, rot[3] = {0, 1, 0};
};
template <>
struct DiagWave<1> {
  static constexpr int NF = 6, NR = 2;
  static constexpr bool ROTC = false;
  static constexpr int frag[6] = {2, 3, 4, 5, 6, 7};
  static constexpr int bi[7] = {0, 0, 0, 1, 1, 0, 0}, bj[7] = {1, 2, 3, 2, 3, 4, 5};
  static constexpr int dg[2] = {0, 1}, rot[3] = {0, 1, 0};
};
template <>
struct DiagWave<2> {
  static constexpr int NF = 5, NR = 3;
  static constexpr bool ROTC = false;
  static constexpr int frag[6] = {1, 4, 5, 6, 7, 0};
  static constexpr int bi[7] = {1, 1, 1, 2, 2, 0, 0}, bj[7] = {2, 3, 4, 3, 4, 1, 2};
  static constexpr int dg[2] = {1, 2}, rot[3] = {0, 1, 2};
};
template <>
struct DiagWave<3> {
  static constexpr int NF = 5, NR = 2;
  static constexpr bool ROTC = true;
  static constexpr int frag[6] = {0, 1, 3, 6, 7, 0};
  static constexpr int bi[7] = {3, 0, 0, 1, 1, 2, 2}, bj[7] = {4, 3, 4, 3, 4, 3, 4};
  static constexpr int dg[2] = {3, 4}, rot[3] = {3, 4, 0};
};

template <int W>
__device__ __forceinline__ void diag_tile(const PackedArgs& a, const TileOut& o, int f, int I,
                                          int t_begin, int t_end, uint8_t* lds) {
  typedef DiagWave<W> D;
  const int tid = threadIdx.x, lane = tid & 63;
  const int ngrain = (t_end - t_begin) / PK_GRAIN;
  const int step_b = a.blocks * BLOCK_BYTES, round_b = 4 * step_b;
  const uint8_t* base = a.packed + ((long long)f * a.steps + t_begin / PK_STEP) * step_b;
  const __amdgpu_buffer_rsrc_t rb = stream_rsrc(base + 2 * I * BLOCK_BYTES);
  // staging: 16-byte units tid + 256 k (k < 12), 768 a step, 384 of either
  // block; a missing second block (odd counts) reads the first again (its
  // results are never written)
  const int second = 2 * I + 1 < a.blocks ? 0 : BLOCK_BYTES;
  int vb[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int e = tid + 256 * k;
    vb[k] = 16 * e - (e < 384 ? 0 : second);
  }
  v16f re[7], im[7], dd[2];
#pragma unroll
  for (int b = 0; b < 7; ++b) re[b] = im[b] = v16f{};
  dd[0] = dd[1] = v16f{};
  v4i st[12];
  auto load_b = [&](int off, int k) { st[k] = ld16(rb, vb[k % 3], off + (k / 3) * step_b); };
  auto stage = [&](uint8_t* d, int k) {
    *reinterpret_cast<v4i*>(d + 16 * (tid + 256 * k)) = st[k];
  };
  // one step: 18 MFMAs of fragments B with rotations R, which the first slots
  // make (see off_tile)
  auto step = [&](auto rd, const v8i (&B)[6], v8i (&Bn)[6], const uint8_t* nu, auto&& extra) {
    constexpr int RD = decltype(rd)::value;
    v8i R[3] = {v8i{}, v8i{}, v8i{}};
#pragma unroll
    for (int k = 0; k < 18; ++k) {
      // seven real blocks, both diagonals' real products, then the others
      const int b = k % 9, i = b < 7 ? D::bi[b] : D::dg[b - 7], j = b < 7 ? D::bj[b] : i;
      int x = 0;
#pragma unroll
      for (int r = 0; r < D::NR; ++r)
        if (D::rot[r] == (D::ROTC ? j : i)) x = r;
      v16f& acc = b >= 7 ? dd[b - 7] : k < 9 ? re[b] : im[b];
      if (k < 9)
        acc = mfma6(B[i], B[j], acc);
      else
        acc = D::ROTC ? mfma6(B[i], R[x], acc) : mfma6(R[x], B[j], acc);
      if (k >= RD && k - RD < 2 * D::NF) {
        const int n = (k - RD) >> 1;
        const uint8_t* u = nu + D::frag[n] * FRAG_BYTES;
        if (((k - RD) & 1) == 0) {
          Bn[n] = op6(lds16(u + 16 * lane), v2i{0, 0});
        } else {
          const v2i hi = lds8(u + 1024 + 8 * lane);
          Bn[n][4] = hi.x;
          Bn[n][5] = hi.y;
        }
      }
      if (k < 3 * D::NR) rot6<D::ROTC>(R[k / 3], B[D::rot[k / 3]], k % 3);
      extra(k);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  v8i B0[6], B1[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) B0[q] = B1[q] = v8i{};
#pragma unroll
  for (int k = 0; k < 12; ++k) load_b(0, k);
#pragma unroll
  for (int k = 0; k < 12; ++k) stage(lds, k);
#pragma unroll
  for (int k = 0; k < 12; ++k) load_b(ngrain > 1 ? round_b : 0, k);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < D::NF; ++q) {
    const uint8_t* u = lds + D::frag[q] * FRAG_BYTES;
    B0[q] = op6(lds16(u + 16 * lane), lds8(u + 1024 + 8 * lane));
  }
  __builtin_amdgcn_sched_barrier(0);
  const std::integral_constant<int, 0> at0;
  const std::integral_constant<int, 4> at4;
  for (int g = 0; g < ngrain; ++g) {
    const uint8_t* cur = lds + (g & 1) * PK_STAGE;
    uint8_t* nxt = lds + ((g + 1) & 1) * PK_STAGE;
    const int ob = min(g + 2, ngrain - 1) * round_b;
    step(at0, B0, B1, cur + 8 * FRAG_BYTES, [&](int) {});
    step(at0, B1, B0, cur + 16 * FRAG_BYTES, [&](int) {});
    step(at0, B0, B1, cur + 24 * FRAG_BYTES, [&](int k) {
      if (k < 12) {
        stage(nxt, k);
        load_b(ob, k);
      }
    });
    step(at4, B1, B0, nxt, [&](int k) {
      if (k == 3) __syncthreads();
    });
  }
  __syncthreads();
  int2* c = reinterpret_cast<int2*>(lds);
  load_corr(a, f, 256 * I, 256, t_begin / a.sumb, (t_end + a.sumb - 1) / a.sumb, c);
  __syncthreads();
  int* m = reinterpret_cast<int*>(lds + 4096) + W * PK_MAT;
  auto blk = [](int i, int j) { return 8 * i - i * (i - 1) / 2 + j - i; };
#pragma unroll
  for (int b = 0; b < 7; ++b) {
    const int i = D::frag[D::bi[b]], j = D::frag[D::bj[b]];
    put_off(o, blk(i, j), 256 * I + 32 * i, 256 * I + 32 * j, re[b], im[b], c + 32 * i, c + 32 * j,
            lane);
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int i = D::frag[D::dg[b]];
    put_diag(o, blk(i, i), 256 * I + 32 * i, dd[b], c + 32 * i, m, lane);
  }
}

}  // namespace

__global__ void __launch_bounds__(256, 1) xcorr_packed_kernel(PackedArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * PK_STAGE];
  const int nhead = a.head_tiles * a.nslices;
  const int b = blockIdx.x;
  int f, p, s, n, item;
  if (b < nhead) {
    const int logical = xcd_logical_id(b, nhead);
    p = logical % a.tiles_per_chan;
    const int rest = logical / a.tiles_per_chan;
    s = rest % a.nslices;
    f = rest / a.nslices;
    n = a.nslices;
    item = (f * a.tiles_per_chan + p) * n + s;
  } else {
    const int rem = a.nchan * a.tiles_per_chan - a.head_tiles;
    const int k = xcd_logical_id(b - nhead, rem * a.tail_slices);
    const int g = a.head_tiles + k % rem;
    s = k / rem;
    f = g / a.tiles_per_chan;
    p = g % a.tiles_per_chan;
    n = a.tail_slices;
    item = (g - a.head_tiles) * n + s;
  }
  const int len = b < nhead ? a.slice_len : a.tail_len;
  int I, J;
  packed_tile_of(p, a.blocks, I, J);
  // uniform: scalar registers, as the buffer resources need them
  f = __builtin_amdgcn_readfirstlane(f);
  I = __builtin_amdgcn_readfirstlane(I);
  J = __builtin_amdgcn_readfirstlane(J);
  const int t_begin = __builtin_amdgcn_readfirstlane(s * len);
  const int t_end = min(a.steps * PK_STEP, t_begin + len);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const long long NB = (long long)a.N * (a.N + 1) / 2;
  TileOut o{a.vis + 2 * (long long)f * NB, n > 1 ? a.partial + (long long)item * PK_PART : nullptr,
            a.N, t_end - t_begin, a.write_mode};
  if (J >= 0) {
    off_tile(a, o, f, I, J, t_begin, t_end, wave, lds);
  } else {
    switch (wave) {
      case 0: diag_tile<0>(a, o, f, I, t_begin, t_end, lds); break;
      case 1: diag_tile<1>(a, o, f, I, t_begin, t_end, lds); break;
      case 2: diag_tile<2>(a, o, f, I, t_begin, t_end, lds); break;
      default: diag_tile<3>(a, o, f, I, t_begin, t_end, lds); break;
    }
  }
}

// Sum the slices' partial blocks of tiles first, first + 1, ... into vis: one
// workgroup per (tile, block).
__global__ void __launch_bounds__(256) packed_reduce_kernel(PackedArgs a, int first, int ns) {
  const int blk = blockIdx.x % 36, t = blockIdx.x / 36, g = first + t;
  const int f = g / a.tiles_per_chan;
  int I, J;
  packed_tile_of(g % a.tiles_per_chan, a.blocks, I, J);
  int i0, j0;
  if (J >= 0) {
    if (blk >= 32) return;
    i0 = 256 * I + 32 * (blk >> 2);
    j0 = 128 * J + 32 * (blk & 3);
  } else {
    int i = 0, k = blk;
    while (k >= 8 - i) k -= 8 - i++;
    i0 = 256 * I + 32 * i;
    j0 = i0 + 32 * k;
  }
  if (i0 >= a.N || j0 >= a.N) return;
  const int2* p = a.partial + (long long)t * ns * PK_PART + (long long)blk * 1024;
  int32_t* base = a.vis + 2LL * f * ((long long)a.N * (a.N + 1) / 2);
  const int lane = threadIdx.x & 63, j = j0 + (lane & 31);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int v = 4 * u + (threadIdx.x >> 6);
    int2 r = make_int2(0, 0);
    for (int s = 0; s < ns; ++s) {
      const int2 w = p[(long long)s * PK_PART + 64 * v + lane];
      r.x += w.x;
      r.y += w.y;
    }
    const int i = i0 + blk_row16(v, lane);
    if (i < a.N && j < a.N && j >= i) {
      int2* q = reinterpret_cast<int2*>(base + 2 * pair_index(i, j, a.N));
      if (a.write_mode == WM_ADD) {
        const int2 w = *q;
        r.x += w.x;
        r.y += w.y;
      }
      *q = r;
    }
  }
}

hipError_t launch_packed(const PackedArgs& a, hipStream_t stream) {
  const long long W = (long long)a.nchan * a.tiles_per_chan;
  const long long grid = (long long)a.head_tiles * a.nslices + (W - a.head_tiles) * a.tail_slices;
  if (grid <= 0) return hipSuccess;
  if (grid > 0x7fffffffLL || (a.steps & 3)) return hipErrorInvalidValue;
  if ((a.nslices > 1 || a.tail_slices > 1) && !a.partial) return hipErrorInvalidValue;
  if (a.nslices > 1 && a.tail_slices > 0) return hipErrorInvalidValue;  // one of the two
  hipLaunchKernelGGL(xcorr_packed_kernel, dim3((unsigned)grid), dim3(256), 0, stream, a);
  const long long sum = a.nslices > 1 ? W : a.tail_slices > 1 ? W - a.head_tiles : 0;
  if (sum * 36 > 0x7fffffffLL) return hipErrorInvalidValue;
  if (sum > 0)
    hipLaunchKernelGGL(packed_reduce_kernel, dim3((unsigned)(sum * 36)), dim3(256), 0, stream, a,
                       (int)(W - sum), a.nslices > 1 ? a.nslices : a.tail_slices);
  return hipGetLastError();
}

}  // namespace xeng
