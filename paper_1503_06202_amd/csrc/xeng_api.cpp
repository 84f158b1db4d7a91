// C ABI of the X-engine (declared in include/xeng.h): plans, argument checks,
// launch configuration and the batched form's work lists and graphs.
//
// Every check that can fail on arguments runs on the host before the first
// HIP call, so those errors are reported the same with or without a GPU.
#include "xeng.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <new>
#include <queue>
#include <string>
#include <vector>

#include "xeng_chan.hpp"
#include "xeng_internal.hpp"
#include "xeng_noalloc.hpp"
#include "xeng_packed.hpp"

namespace {

constexpr int kTile = 128;   // tile edge of the kernels
constexpr int kChunk = 64;   // samples per staged chunk
constexpr int kOccupancy = 2;  // workgroups per CU (LDS: 64 KiB each)
constexpr int kChanMax = 2 * kTile;  // inputs of the channel kernel
// Output gating: extra work gates one launch segment can need when gates are
// split (fewer than 2 x 64 = 128; see xeng_correlate_gated).
constexpr int kSplitMax = 128;
// Packed path: device memory of a plan's operands, at most (a channel that
// takes more on its own gets what it needs); larger frames run in groups of
// channels.
constexpr size_t kPackedMax = 4ull << 30;
// Partial outputs of a slice count that the plan names, at most; more take the
// tile kernels, whose slices add into vis (16 slices of 2048 inputs and 16
// channels would store 5.4 GB, of 128 inputs and 1024 channels 1.1 GB).  The
// automatic counts stay below it.
constexpr size_t kPartMax = 1ull << 30;
// Calls that do without a workspace after its memory was refused, before one
// asks again: a refusal costs more than many a frame.
constexpr int kRefusedCalls = 64;
constexpr int kStageRing = 4;  // pinned staging copies of a batch plan's instance table

enum PlanKind { PLAN_SINGLE = 1, PLAN_BATCH = 2 };

}  // namespace

struct xeng_plan_s {
  int kind = 0;
  int N = 0, F = 0, T_max = 0;
  unsigned flags = 0;
  int form = XENG_FORM_I8;
  bool accumulate = false;
  int split_t = 0;  // 0 = automatic
  int kernel = 0;   // 0 = automatic (packed path included), 1 = 128 x 128 tiles, 2 = 128 x 256 tiles,
                    // 3 / 4 = 128 x 128 tiles with split / common diagonal roles
  bool once = false;  // see xeng_plan_once
  int cu_count = 0;
  std::string err;

  // batched form
  std::vector<xeng_instance> insts;
  std::vector<xeng::BatchItem> items;
  std::vector<int> inst_zero;
  bool any_zero = false;
  // pinned staging of the instance table: a ring of kStageRing copies, so
  // that a call refills one while earlier calls' uploads are still queued
  xeng::BatchInst* h_insts = nullptr;
  xeng::BatchInst* d_insts = nullptr;
  xeng::BatchItem* d_items = nullptr;
  int* d_counter = nullptr;
  hipEvent_t copy_done[kStageRing] = {};
  bool copy_pending[kStageRing] = {};
  int stage_next = 0;
  std::vector<const void*> uploaded;  // pointers now in d_insts
  hipGraphExec_t graph_exec = nullptr;
  hipStream_t capture_stream = nullptr;
  // instances that calls take by the packed path, and a plan of the others
  // (or nullptr, if there are none)
  std::vector<int> large;
  xeng_plan_t rest = nullptr;

  // output gating (xeng_plan_gated): run tables, pinned staging and device
  int G_max = 0;
  long long gate_off_cap = 0, runs_cap = 0, vgate_cap = 0;  // entries
  int* h_gate_off = nullptr;
  int2* h_runs = nullptr;
  int2* h_vgate = nullptr;
  int* d_gate_off = nullptr;
  int2* d_runs = nullptr;
  int2* d_vgate = nullptr;
  hipEvent_t gate_done = nullptr;
  bool gate_pending = false;
  std::vector<int> gate_count, gate_fill;  // host work space of the run tables, G_max each
  std::vector<int> gate_zero;              // gates to clear before a split gate adds into them
  std::vector<int> seg_goff, seg_nvg;      // per launch segment: first table entry, work gates

  // workspace of the calls that need one (partial outputs of time slices,
  // packed operands): plan-owned, grown on demand; see workspace()
  uint8_t* d_ws = nullptr;
  size_t ws_bytes = 0;
  int ws_device = 0;
  // the size last refused for want of memory, asked for again after kRefusedCalls calls
  size_t ws_refused = SIZE_MAX;
  int ws_skipped = 0;
  bool ws_pending = false;        // a call has used it
  hipEvent_t ws_used = nullptr;   // recorded after every use; NULL while all were on the null stream

  // time shifting (xeng_plan_set_delays): per-segment delays and block maxima
  bool shift = false;
  int* d_seg_delay = nullptr;
  int* d_blk_delay = nullptr;
  // delays that differ inside a 128-input block: shifted copy of the frame
  bool shift_copy = false;
  int shift_max = 0;  // the largest delay
  uint8_t* d_shifted = nullptr;

  // flagged data (xeng_plan_flagged): event frame, its correlation and counters
  bool flagged = false;
  long long flag_cap = 0;  // event rows per channel
  int flag_nseg = 0;       // launch segments of the event correlation
  uint8_t* d_fU = nullptr;
  int32_t* d_fX = nullptr;
  int* d_fint = nullptr;   // cnt [F], single [F N], n [F N], R [1], gate_off [2 nseg]
  int2* d_fruns = nullptr;

  // The delay tables and the beam weight operands are replaced only after the
  // plan's last call that reads them has finished (a plan has at most one
  // call in flight): that call records tables_used on its stream.
  hipEvent_t tables_used = nullptr;
  bool tables_pending = false;

  // discrete beamforming (xeng_plan_beams): weight operands and offset terms
  int B = 0, beam_S = 0, beam_nbt = 0;
  bool beams_ready = false;
  void* d_wop = nullptr;
  int* d_bcorr = nullptr;
};

namespace {

int hip_fail(xeng_plan_t p, hipError_t e, const char* what) {
  if (p) {
    p->err = std::string(what) + ": " + hipGetErrorName(e) + " (" + hipGetErrorString(e) + ")";
  }
  return XENG_EHIP;
}

// Create the plan's tables_used event if needed, and wait until the plan's
// last call that read its delay or weight tables has finished.
hipError_t wait_tables(xeng_plan_t p) {
  if (!p->tables_used) return hipEventCreateWithFlags(&p->tables_used, hipEventDisableTiming);
  if (!p->tables_pending) return hipSuccess;
  const hipError_t e = hipEventSynchronize(p->tables_used);
  if (e == hipSuccess) p->tables_pending = false;
  return e;
}

// After a call that read the tables: mark them in use until `s` gets here.
int mark_tables(xeng_plan_t p, hipStream_t s) {
  const hipError_t e = hipEventRecord(p->tables_used, s);
  if (e != hipSuccess) return hip_fail(p, e, "hipEventRecord");
  p->tables_pending = true;
  return XENG_OK;
}

bool flags_ok(unsigned flags, bool batch = false) {
  const unsigned form = flags & XENG_FORM_MASK;
  if (form != XENG_FORM_I8 && form != XENG_FORM_F8) return false;
  unsigned known = XENG_FORM_MASK | XENG_ACCUMULATE;
  if (batch) {
    known |= XENG_SHARED_VIS;
    if ((flags & XENG_SHARED_VIS) && !(flags & XENG_ACCUMULATE)) return false;
  }
  return (flags & ~known) == 0;
}

int ensure_cu_count(xeng_plan_t p) {
  if (p->cu_count > 0) return XENG_OK;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(p, e, "hipGetDevice");
  int cus = 0;
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return hip_fail(p, e, "hipDeviceGetAttribute");
  p->cu_count = cus > 0 ? cus : 1;
  return XENG_OK;
}

long long tiles_per_channel(int N) {
  const long long nt = (N + kTile - 1) / kTile;
  return nt * (nt + 1) / 2;
}

// Fast loads: 16-byte row pieces at any alignment, with per-lane offsets (64
// rows) that fit 31 bits.
bool fast_loads(int F, int N) { return (long long)F * N <= (1LL << 25); }

// 128 x 256 tiles (I, J) with J >= I / 2.
long long wide_tiles_per_channel(int N) {
  const long long nI = (N + kTile - 1) / kTile, nJ = (N + 2 * kTile - 1) / (2 * kTile);
  long long t = 0;
  for (long long I = 0; I < nI; ++I) t += nJ - I / 2;
  return t;
}

// Time slices per tile.  With W tiles and `slots` resident workgroups, S
// slices take round_cost(W S) rounds of 1/S of the work each; every extra
// slice costs about 4% more (exact int32 atomic adds into vis, which must be
// cleared first).  auto_slices picks the S that minimises round_cost(W S) /
// S * (1 + 0.04 (S - 1)), keeping slices of at least 1024 samples.
//
// round_cost: rounds of resident workgroups that `items` work items take on
// `slots` slots (`occupancy` per CU).  A last round that leaves each CU at
// most one workgroup costs less than a full one, since that workgroup has the
// CU to itself: on 192 tiles at N = 256 (512 slots) the timings of 1 to 8
// slices fit a cost of about 0.6 round for it.
constexpr double kLoneRound = 0.6;
double round_cost(long long items, long long slots, int occupancy) {
  const long long full = items / slots, rem = items % slots;
  if (rem == 0) return (double)full;
  return (double)full + (occupancy > 1 && rem * occupancy <= slots ? kLoneRound : 1.0);
}

double slice_cost(long long tiles, int S, long long slots, int occupancy) {
  return round_cost(tiles * S, slots, occupancy) / S * (1.0 + 0.04 * (S - 1));
}

int auto_slices(long long tiles, int T, int cu_count, int occupancy = kOccupancy) {
  const long long slots = (long long)cu_count * occupancy;
  const int smax = std::max(1, std::min(16, T / 1024));
  int best = 1;
  double best_cost = 1e300;
  for (int S = 1; S <= smax; ++S) {
    const double cost = slice_cost(tiles, S, slots, occupancy);
    if (cost < best_cost - 1e-12) {
      best_cost = cost;
      best = S;
    }
  }
  return best;
}

// Samples one launch of the 128 x 128 kernels may integrate (sums of codes
// stay exact: f32 below 2^24, int32 below 2^31).
int segment_max(int form) { return form == XENG_FORM_F8 ? XENG_F8_FLUSH_MAX : XENG_I8_SEG_MAX; }

// Time slices of a batch instance: S slices of `len` samples (a multiple of
// kChunk), from its split_t or else the batch's automatic count s_auto; no
// slice integrates more than segment_max(form) samples.
void batch_slices(const xeng_instance& d, int s_auto, int form, int& S, int& len) {
  S = d.split_t > 0 ? d.split_t : std::max(1, std::min(s_auto, d.T / 1024));
  const int seg_max = segment_max(form);
  S = std::max(S, (d.T + seg_max - 1) / seg_max);
  S = std::min(S, (d.T + kChunk - 1) / kChunk);
  len = (d.T + S - 1) / S;
  len = (len + kChunk - 1) / kChunk * kChunk;
  S = (d.T + len - 1) / len;
}

// Compute units of the current device for a plan being built; without a
// device (plans can be built and validated on a host with no GPU) the count
// of an MI355X.  Only the automatic slice count depends on it.
int cu_count_hint() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus < 1) {
    (void)hipGetLastError();
    return 256;
  }
  return cus;
}

}  // namespace

extern "C" {

int xeng_version(void) { return (1 << 16) | 0; }

const char* xeng_strerror(int code) {
  switch (code) {
    case XENG_OK: return "success";
    case XENG_EINVAL: return "invalid argument";
    case XENG_EPLAN: return "argument does not match the plan";
    case XENG_EOVERFLOW: return "integration too long for exact int32 sums";
    case XENG_EHIP: return "HIP runtime or launch error";
    case XENG_ENOMEM: return "out of memory";
    case XENG_ELIMIT: return "request exceeds the fixed workspace of the allocation-free entry point";
    default: return "unknown error code";
  }
}

int xeng_plan(xeng_plan_t* out, int N, int F, int T_max, unsigned flags) {
  if (!out) return XENG_EINVAL;
  *out = nullptr;
  if (N < 1 || F < 1 || T_max < 1 || N > XENG_N_MAX || !flags_ok(flags)) return XENG_EINVAL;
  if (T_max > XENG_T_EXACT_MAX) return XENG_EOVERFLOW;
  xeng_plan_t p = new (std::nothrow) xeng_plan_s();
  if (!p) return XENG_ENOMEM;
  p->kind = PLAN_SINGLE;
  p->N = N;
  p->F = F;
  p->T_max = T_max;
  p->flags = flags;
  p->form = (int)(flags & XENG_FORM_MASK);
  p->accumulate = (flags & XENG_ACCUMULATE) != 0;
  *out = p;
  return XENG_OK;
}

int xeng_plan_gated(xeng_plan_t* out, int N, int F, int T_max, int G_max, unsigned flags) {
  if (!out) return XENG_EINVAL;
  *out = nullptr;
  if (G_max < 1 || G_max > XENG_G_MAX) return XENG_EINVAL;
  xeng_plan_t p = nullptr;
  int rc = xeng_plan(&p, N, F, T_max, flags);
  if (rc != XENG_OK) return rc;
  const int seg = segment_max(p->form);
  const long long nseg = (T_max + seg - 1) / seg;
  p->G_max = G_max;
  try {
    p->gate_count.assign(G_max, 0);
    p->gate_fill.assign(G_max, 0);
    p->gate_zero.assign(G_max, 0);
    p->seg_goff.assign(nseg, 0);
    p->seg_nvg.assign(nseg, 0);
  } catch (const std::bad_alloc&) {
    xeng_destroy(p);
    return XENG_ENOMEM;
  }
  // A segment has at most G_max + kSplitMax work gates (see xeng_correlate_gated).
  p->vgate_cap = nseg * ((long long)G_max + kSplitMax);
  p->gate_off_cap = p->vgate_cap + nseg;
  p->runs_cap = (long long)T_max + nseg;  // at most one run per sample, plus a cut per segment
  hipError_t e = hipHostMalloc((void**)&p->h_gate_off, p->gate_off_cap * sizeof(int),
                               hipHostMallocDefault);
  if (e == hipSuccess)
    e = hipHostMalloc((void**)&p->h_runs, p->runs_cap * sizeof(int2), hipHostMallocDefault);
  if (e == hipSuccess)
    e = hipHostMalloc((void**)&p->h_vgate, p->vgate_cap * sizeof(int2), hipHostMallocDefault);
  if (e == hipSuccess) e = hipMalloc((void**)&p->d_gate_off, p->gate_off_cap * sizeof(int));
  if (e == hipSuccess) e = hipMalloc((void**)&p->d_runs, p->runs_cap * sizeof(int2));
  if (e == hipSuccess) e = hipMalloc((void**)&p->d_vgate, p->vgate_cap * sizeof(int2));
  if (e == hipSuccess) e = hipEventCreateWithFlags(&p->gate_done, hipEventDisableTiming);
  if (e != hipSuccess) {
    rc = e == hipErrorOutOfMemory ? XENG_ENOMEM : XENG_EHIP;
    (void)hipGetLastError();
    xeng_destroy(p);
    return rc;
  }
  *out = p;
  return XENG_OK;
}

int xeng_plan_set_delays(xeng_plan_t p, const int32_t* delays, int D_max) {
  if (!p) return XENG_EINVAL;
  if (p->kind != PLAN_SINGLE) return XENG_EPLAN;
  if (!delays) {
    p->shift = false;
    return XENG_OK;
  }
  const int N = p->N, nseg = (N + 15) / 16, nt = (N + kTile - 1) / kTile;
  if (D_max < 0 || ((long long)D_max + 64) * p->F * N >= (1LL << 31)) return XENG_EINVAL;
  std::vector<int> seg(nseg), blk(nt, 0);
  for (int n = 0; n < N; ++n) {
    if (delays[n] < 0 || delays[n] > D_max) return XENG_EINVAL;
    if (delays[n] != delays[n & ~15]) return XENG_EINVAL;  // one delay per 16-input segment
  }
  for (int k = 0; k < nseg; ++k) {
    seg[k] = delays[16 * k];
    blk[(16 * k) / kTile] = std::max(blk[(16 * k) / kTile], seg[k]);
  }
  // Uniform delays within every 128-input block are applied in the kernels'
  // loads; otherwise the frame is copied, shifted, into plan-owned memory.
  bool fine = false;
  for (int k = 0; k < nseg; ++k) fine |= seg[k] != blk[(16 * k) / kTile];
  // the plan's last call may still read the old delays
  hipError_t e = wait_tables(p);
  if (e == hipSuccess && fine && !p->d_shifted)
    e = hipMalloc((void**)&p->d_shifted, (size_t)p->T_max * p->F * N);
  if (e == hipSuccess && !p->d_seg_delay) e = hipMalloc((void**)&p->d_seg_delay, nseg * sizeof(int));
  if (e == hipSuccess && !p->d_blk_delay) e = hipMalloc((void**)&p->d_blk_delay, nt * sizeof(int));
  if (e == hipSuccess)
    e = hipMemcpy(p->d_seg_delay, seg.data(), nseg * sizeof(int), hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(p->d_blk_delay, blk.data(), nt * sizeof(int), hipMemcpyHostToDevice);
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? XENG_ENOMEM : hip_fail(p, e, "delay upload");
  p->shift = true;
  p->shift_copy = fine;
  p->shift_max = *std::max_element(seg.begin(), seg.end());
  return XENG_OK;
}

int xeng_plan_set_tuning(xeng_plan_t p, int split_t, int kernel) {
  if (!p || split_t < 0 || kernel < 0 || kernel > 5) return XENG_EINVAL;
  p->split_t = split_t;
  p->kernel = kernel;
  return XENG_OK;
}

const char* xeng_plan_error(xeng_plan_t p) { return p ? p->err.c_str() : ""; }

// Whether `s` is being captured into a HIP graph (or cannot be asked): such a
// call takes the kernels that need no plan-owned workspace, which a later call
// could replace or overwrite between the graph's replays.
static bool stream_captures(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return st != hipStreamCaptureStatusNone;
}

// While it lives, this thread may allocate, free and wait although another
// stream is being captured, here or in another thread (a capture in the default
// mode refuses that to all threads): none of it concerns that capture.
struct BesideCaptures {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  bool set = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  BesideCaptures() = default;
  BesideCaptures(const BesideCaptures&) = delete;
  ~BesideCaptures() {
    if (set) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

// Record the workspace's event on `s`.
static int workspace_record(xeng_plan_t p, hipStream_t s) {
  hipError_t e = hipSuccess;
  if (!p->ws_used) e = hipEventCreateWithFlags(&p->ws_used, hipEventDisableTiming);
  if (e != hipSuccess) return hip_fail(p, e, "hipEventCreate");
  e = hipEventRecord(p->ws_used, s);
  return e == hipSuccess ? XENG_OK : hip_fail(p, e, "hipEventRecord");
}

// The plan's workspace, at least `bytes`, for a call on `s`: grown when needed
// (after the plan's last call that used it), and ordered after that call.
// Every use records an event that the next one waits for on its stream, except
// while all uses are on the null stream, which orders them itself and is never
// destroyed: an event is a good part of a small frame's call (N = 64, F = 4, T =
// 8192: 14.8 us with, 12.0 without).  The first use on another stream records
// the event for those before it.  An equal handle says nothing
// on other streams: hipStreamPerThread is another one in every thread, and the
// handles of destroyed streams are given out again.
// XENG_ENOMEM: the call has to do without (no memory, a stream of another device
// than the memory's, or its order after the null stream cannot be had while
// another stream's capture includes that one).
static int workspace(xeng_plan_t p, size_t bytes, hipStream_t s) {
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return hip_fail(p, e, "hipGetDevice");
  if (s != nullptr) {
    hipDevice_t own = device;
    if (hipStreamGetDevice(s, &own) != hipSuccess) (void)hipGetLastError();
    if (own != device) return XENG_ENOMEM;
  }
  if (p->d_ws && device != p->ws_device) return XENG_ENOMEM;
  if (p->ws_pending && !p->ws_used && s != nullptr) {
    if (stream_captures(nullptr)) return XENG_ENOMEM;
    const int rc = workspace_record(p, nullptr);
    if (rc != XENG_OK) return rc;
  }
  if (bytes > p->ws_bytes) {
    if (bytes >= p->ws_refused && ++p->ws_skipped < kRefusedCalls) return XENG_ENOMEM;
    const BesideCaptures relaxed;
    // the new memory first: a plan that cannot grow keeps what it has
    uint8_t* grown = nullptr;
    e = hipMalloc((void**)&grown, bytes);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      if (e != hipErrorOutOfMemory) return hip_fail(p, e, "hipMalloc (workspace)");
      p->ws_refused = bytes;
      p->ws_skipped = 0;
      return XENG_ENOMEM;
    }
    if (p->ws_pending) {
      e = p->ws_used ? hipEventSynchronize(p->ws_used) : hipStreamSynchronize(nullptr);
      if (e != hipSuccess) {
        (void)hipFree(grown);
        return hip_fail(p, e, "workspace synchronization");
      }
      p->ws_pending = false;
    }
    if (p->d_ws) (void)hipFree(p->d_ws);
    p->d_ws = grown;
    p->ws_device = device;
    p->ws_bytes = bytes;
    p->ws_refused = SIZE_MAX;
  } else if (p->ws_pending && p->ws_used) {
    e = hipStreamWaitEvent(s, p->ws_used, 0);
    if (e != hipSuccess) return hip_fail(p, e, "hipStreamWaitEvent");
  }
  return XENG_OK;
}

// After the last kernel of a call that may use the workspace, also where a
// later launch of the call failed.
static int workspace_used(xeng_plan_t p, hipStream_t s) {
  p->ws_pending = true;
  return s != nullptr || p->ws_used ? workspace_record(p, s) : XENG_OK;
}

// The packed path (xeng_packed.hpp): bytes of one channel's operands and code
// sums (at most) over `len` samples.
static size_t packed_channel_bytes(int N, int len) {
  const size_t steps = 4 * (size_t)((len + xeng::PK_GRAIN - 1) / xeng::PK_GRAIN);
  const size_t blocks = (N + kTile - 1) / kTile;
  const size_t nsum = (steps * xeng::PK_STEP + xeng::PK_SUMB_SHORT - 1) / xeng::PK_SUMB_SHORT;
  return steps * blocks * xeng::BLOCK_BYTES + nsum * blocks * kTile * sizeof(int2);
}

// The slice count that a plan names for its frames (batch plans name theirs per
// instance, and those keep the tiles), or 0.
static int named_slices(xeng_plan_t p) { return p->kind == PLAN_SINGLE ? p->split_t : 0; }

// The packed path's schedule for W tiles of `plen` samples on `cus` compute
// units (one workgroup each): uniform slices, or R full rounds of whole tiles
// and the rest in slices that fill one more round.
struct PackedSchedule {
  int nslices, slice_len;
  long long head;
  int tail_slices, tail_len;
};

static PackedSchedule packed_schedule(long long W, int plen, int sumb, int cus, int split_t) {
  auto round_slice = [&](int n) {
    const int l = (plen + n - 1) / n;
    return (l + sumb - 1) / sumb * sumb;
  };
  PackedSchedule c{1, plen, W, 0, 0};
  if (split_t > 0) {
    c.slice_len = round_slice(split_t);
    c.nslices = (plen + c.slice_len - 1) / c.slice_len;
    return c;
  }
  // microseconds: a step of a tile, the start and end of a round, and what a
  // sliced item adds (its partial blocks written and read back)
  const double step = 0.42, round = 12.0, fixed = 10.0, item = 0.10;
  const double steps = plen / (double)xeng::PK_STEP;
  auto rounds = [&](long long n) { return (double)((n + cus - 1) / cus); };
  double best = rounds(W) * (steps * step + round);
  const int smax = std::min(16, plen / sumb);
  for (int S = 2; S <= smax; ++S) {
    const int sl = round_slice(S), n = (plen + sl - 1) / sl;
    if (n != S) continue;
    const double t = rounds(W * n) * (sl / (double)xeng::PK_STEP * step + round) + fixed + item * W * n;
    if (t < best) {
      best = t;
      c.nslices = n;
      c.slice_len = sl;
    }
  }
  const long long R = W / cus, rem = W - R * cus;
  if (R > 0 && rem > 0) {
    for (int S = 2; S <= smax; ++S) {
      const int sl = round_slice(S), n = (plen + sl - 1) / sl;
      if (n != S) continue;
      const double t = R * (steps * step + round) +
                       rounds(rem * n) * (sl / (double)xeng::PK_STEP * step + round) + fixed +
                       item * rem * n;
      if (t < best) {
        best = t;
        c.nslices = 1;
        c.slice_len = plen;
        c.head = R * cus;
        c.tail_slices = n;
        c.tail_len = sl;
      }
    }
  }
  return c;
}

// The tile kernels' schedule of W tiles over len samples: uniform slices (the
// count named, or auto_slices'), or a head/tail split: R full rounds of whole
// tiles (plain stores or adds), then the remaining tiles cut into slices that
// fill one more round (atomic adds into a cleared region), if the cost model of
// auto_slices prefers it.
struct TileSchedule {
  int nslices, slice_len;
  long long head;
  int tail_slices, tail_len;
};

static TileSchedule tile_schedule(long long W, int len, int cus, int occupancy, int split_t,
                                  bool wide) {
  auto round_chunk = [](int l) { return (l + kChunk - 1) / kChunk * kChunk; };
  int n = split_t > 0 ? split_t : auto_slices(W, len, cus, occupancy);
  n = std::min(n, (len + kChunk - 1) / kChunk);
  const int sl = round_chunk((len + n - 1) / n);
  TileSchedule c{(len + sl - 1) / sl, sl, W, 0, 0};
  const long long slots = (long long)cus * occupancy;
  if (split_t == 0 && !wide && W > slots && W % slots != 0 && slots % 8 == 0) {
    const long long R = W / slots, rem = W - R * slots;
    const int smax = std::max(1, std::min(16, len / 1024));
    int St = (int)std::min<long long>(smax, std::max<long long>(1, (slots + rem / 2) / rem));
    const int tl = round_chunk((len + St - 1) / St);
    St = (len + tl - 1) / tl;
    const double cost_tail = (double)R + slice_cost(rem, St, slots, occupancy);
    if (St > 1 && cost_tail < slice_cost(W, c.nslices, slots, occupancy) - 1e-9)
      c = TileSchedule{1, len, R * slots, St, tl};
  }
  return c;
}

static int packed_sumb(int blocks, int nchan, int plen, int cus) {
  const long long wgs = (long long)blocks * nchan *
                        ((plen + xeng::PK_SUMB_LONG - 1) / xeng::PK_SUMB_LONG);
  return wgs >= 4LL * cus ? xeng::PK_SUMB_LONG : xeng::PK_SUMB_SHORT;
}

// Estimated microseconds of one launch of either path (F channels, len samples;
// add: into vis).  Fitted to 1300 frames of 640..4096 inputs, 1..48 channels and
// 1024..40000 samples, both paths timed on each: 5.4% (tiles) and 5.7% (packed)
// rms.  A round's last, partial wave counts as in round_cost, but 0.65 of a round
// for lone workgroups and, after full rounds, three tenths in proportion to its
// size; stores and atomic adds hide behind long items (half of them at 4000
// samples).
static double tiles_us(int N, int F, int len, bool add, int cus) {
  const long long W = tiles_per_channel(N) * F, slots = (long long)cus * kOccupancy;
  const TileSchedule c = tile_schedule(W, len, cus, kOccupancy, 0, false);
  const double mb = 4e-6 * F * N * (N + 1.0);  // visibilities
  auto rounds = [&](long long items) {
    const long long full = items / slots, rem = items % slots;
    double part = rem == 0 ? 0.0 : rem * kOccupancy <= slots ? 0.65 : 1.0;
    if (full > 0) part = 0.3 * rem / slots + 0.7 * part;
    return full + part;
  };
  auto shown = [](double samples) { return 4000.0 / (4000.0 + samples); };
  double samples, stored = 0.0, added = 0.0;
  if (c.tail_slices > 0) {
    const double part = (double)(W - c.head) / W;
    samples = (double)(c.head / slots) * len + rounds((W - c.head) * c.tail_slices) * c.tail_len;
    stored = mb * (1.0 - part) * shown(len);
    added = mb * part * c.tail_slices * shown(c.tail_len);
  } else {
    samples = rounds(W * c.nslices) * c.slice_len;
    (c.nslices > 1 ? added : stored) = mb * c.nslices * shown(c.slice_len);
  }
  return 8.2 + 0.0210 * samples + (add ? 0.282 : 0.1185) * stored + 1.457 * added +
         (c.nslices > 1 ? 2.4 : 0.0) + 0.0765 * mb;
}

static double packed_us(int N, int F, int len, bool add, int cus) {
  const int blocks = (N + kTile - 1) / kTile;
  const int plen = (len + xeng::PK_GRAIN - 1) / xeng::PK_GRAIN * xeng::PK_GRAIN;
  const long long W = (long long)xeng::packed_tiles(blocks) * F;
  const PackedSchedule c = packed_schedule(W, plen, packed_sumb(blocks, F, plen, cus), cus, 0);
  auto rounds = [&](long long items) { return (double)((items + cus - 1) / cus); };
  const double head = rounds(c.head * c.nslices);
  const double tail = c.tail_slices > 0 ? rounds((W - c.head) * c.tail_slices) : 0.0;
  const long long sliced = c.nslices > 1      ? W * c.nslices
                           : c.tail_slices > 0 ? (W - c.head) * c.tail_slices
                                               : 0;
  const double mb = 4e-6 * F * N * (N + 1.0);
  return 7.1 + (0.374 / xeng::PK_STEP) * (head * c.slice_len + tail * c.tail_len) +
         16.6 * (head + tail) + 0.434e-6 * plen * F * blocks * kTile + 0.031 * mb +
         (add ? 0.289 * mb : 0.0) + 0.038 * sliced;
}

// The same for a frame of T samples in launches of at most seg; later ones add.
static double frame_us(double (*us)(int, int, int, bool, int), int N, int F, int T, bool add,
                       int seg, int cus) {
  const int full = T / seg, rest = T % seg;
  const double t =
      full > 0 ? us(N, F, seg, add, cus) + (full - 1) * us(N, F, seg, true, cus) : 0.0;
  return rest > 0 ? t + us(N, F, rest, add || full > 0, cus) : t;
}

static double packed_frame_us(int N, int F, int T, bool add, int cus) {
  return frame_us(packed_us, N, F, T, add, XENG_F8_FLUSH_MAX, cus);
}

// When the packed path is chosen (tuning kernel 0): where its estimate is the
// lower one, by 3% for the estimates' errors.  Packing moves 2.5 bytes of HBM
// traffic a sample (0.52 ms for a GiB of samples) and the FP6 correlation runs
// at about 1.8 times the rate of the int8 tiles, so it pays from about 700 inputs
// on; its three launches, and visibilities that bind short integrations alike,
// leave the tiles ahead on small frames.  Microseconds, tile kernels / packed path:
//   N = 2048, F = 16, T = 32768  3275 / 2372    N = 512, F = 16, T = 32768  258 / 281
//   N = 1024, F = 16, T = 32768   862 / 718     N = 1024, F = 1, T = 8192    63 / 49
//   N = 768,  F = 1, T = 32768     79 / 71      N = 768,  F = 1, T = 8192    45 / 50
//   N = 1426, F = 2, T = 1577 39 / 60   N = 1152, F = 25, T = 1728 113 / 127
//   N = 976, F = 41, T = 2944 229 / 288 N = 1281, F = 2, T = 2600   68 / 59
// Of 800 other frames, drawn alike, 22 run more than 1% slower than on the tiles
// for it, 1.12 times at most; lines in the size alone (2560 samples, or 1536 where
// the tiles' last wave leaves a tenth of the slots unused) had 130 of 1300, up to
// 1.55 times.  Below 230,000 tile-samples (128 x 128 tiles x samples) the
// estimates are not close enough.
// Delays that differ inside a block of 128 inputs (dmax, the largest; else -1)
// cost the tile kernels a copy of the frame that fetches every line eight times
// (1.39 ms for a GiB of 2048 inputs), and the packed path only a longer packing
// pass (0.93 ms): there it pays from 128 inputs on,
//   N = 128, F = 16, T = 32768  131 / 110    N = 384, F = 64, T = 4096   259 / 130
//   N = 512, F = 4,  T = 8192 (328,000)  80 / 64    N = 512, F = 1, T = 32768 (328,000)  76 / 81
// from 340,000 tile-samples and 1536 samples, where its estimate is the lower one
// (N = 224, F = 57, T = 2043, D = 13737, accumulated 78 / 103; N = 144, F = 6, T =
// 28605 69 / 83).  The estimates fit 274 frames of 128..2048 inputs (packed 5%,
// tiles 7% rms; the copy costs three times as much where rows are not aligned): 2
// of them are more than 1% slower for it, 10 by the sizes alone.
static bool packed_pays(int N, int F, int T, int dmax, int form, bool add, int cus) {
  const long long work = tiles_per_channel(N) * F * T;
  if (dmax < 0 ? N <= 640 || T < 1024 || work < 230000 : N < 128 || T < 1536 || work < 340000)
    return false;
  const double packed = packed_frame_us(N, F, T, add, cus);
  const double tiles = frame_us(tiles_us, N, F, T, add, segment_max(form), cus);
  if (dmax < 0) return packed < 0.97 * tiles;
  const double mb = 1e-6 * N * F * T;  // samples, and those that packing reads
  const double read = 1e-6 * ((N + kTile - 1) / kTile * kTile) * F * ((double)T + dmax);
  const double copy = 0.78 + (N % 16 != 0 ? 1.64 : 0.0) + (dmax > 2000 ? 0.25 : 0.0);
  return 8.7 + 0.070 * mb + 0.136 * read + 0.93 * packed < 2.9 + copy * mb + 1.05 * tiles;
}

// Workspace of a packed call: channels per group, operands and partial blocks
// (the largest schedule of the call).
struct PackedNeed {
  int group;
  size_t operands, part;
};

static PackedNeed packed_need(xeng_plan_t p, int N, int F, int T) {
  const int blocks = (N + kTile - 1) / kTile, tpc = xeng::packed_tiles(blocks);
  const int seg = XENG_F8_FLUSH_MAX, seg_len = std::min(T, seg);
  const size_t per_chan = packed_channel_bytes(N, seg_len);
  const int group = (int)std::max<size_t>(1, std::min<size_t>(F, kPackedMax / per_chan));
  size_t part = 0;
  for (int k = 0; k < 4; ++k) {
    const int len = k & 1 ? T % seg : seg_len, nch = k & 2 ? F % group : group;
    if (len == 0 || nch == 0) continue;
    const int plen = (len + xeng::PK_GRAIN - 1) / xeng::PK_GRAIN * xeng::PK_GRAIN;
    const PackedSchedule c =
        packed_schedule((long long)tpc * nch, plen, packed_sumb(blocks, nch, plen, p->cu_count),
                        p->cu_count, named_slices(p));
    const long long items = c.nslices > 1 ? c.head * c.nslices
                                          : ((long long)tpc * nch - c.head) * c.tail_slices;
    part = std::max(part, (size_t)items * xeng::PK_PART * sizeof(int2));
  }
  return PackedNeed{group, (per_chan * group + 255) / 256 * 256, part};
}

// Queue the packed path: per segment of at most XENG_F8_FLUSH_MAX samples and
// group of channels that fits the workspace, pack the samples and correlate the
// packed operands.
static int launch_packed_path(xeng_plan_t p, const PackedNeed& need, const uint8_t* samples, int N,
                              int F, int T, int32_t* vis, hipStream_t s) {
  const int blocks = (N + kTile - 1) / kTile, tpc = xeng::packed_tiles(blocks);
  const int seg = XENG_F8_FLUSH_MAX;
  const auto [group, operands, part] = need;
  hipError_t e = hipSuccess;
  const long long row = (long long)F * N, NB2 = (long long)N * (N + 1);
  const bool aligned = (N % 16 == 0) && ((reinterpret_cast<uintptr_t>(samples) & 15) == 0);
  for (int t0 = 0; t0 < T; t0 += seg) {
    const int len = std::min(seg, T - t0);
    const bool add = p->accumulate || t0 > 0;
    for (int f0 = 0; f0 < F; f0 += group) {
      const int nch = std::min(group, F - f0);
      xeng::PackArgs k;
      k.samples = samples + (long long)f0 * N;
      k.frame_end = samples + (long long)T * row;
      k.N = N;
      k.nchan = nch;
      k.t0 = t0;
      k.t1 = t0 + len;
      k.row_stride = row;
      k.blocks = blocks;
      k.steps = 4 * ((len + xeng::PK_GRAIN - 1) / xeng::PK_GRAIN);
      const int plen = k.steps * xeng::PK_STEP;
      k.sumb = packed_sumb(blocks, nch, plen, p->cu_count);
      k.nsum = (plen + k.sumb - 1) / k.sumb;
      k.packed = p->d_ws;
      k.sums = reinterpret_cast<int2*>(p->d_ws +
                                       (size_t)nch * k.steps * blocks * xeng::BLOCK_BYTES);
      // delays that differ inside a block: by source windows
      k.seg_delay = p->shift ? p->d_seg_delay : nullptr;
      k.dmax = p->shift && p->shift_copy ? p->shift_max : -1;
      k.win = k.sumb;
      e = xeng::launch_pack(k, aligned, s);
      if (e != hipSuccess) return hip_fail(p, e, "pack launch");

      const PackedSchedule c =
          packed_schedule((long long)tpc * nch, plen, k.sumb, p->cu_count, named_slices(p));
      xeng::PackedArgs a;
      a.packed = k.packed;
      a.sums = k.sums;
      a.vis = vis + f0 * NB2;
      a.partial = part ? reinterpret_cast<int2*>(p->d_ws + operands) : nullptr;
      a.N = N;
      a.nchan = nch;
      a.steps = k.steps;
      a.blocks = blocks;
      a.nsum = k.nsum;
      a.sumb = k.sumb;
      a.tiles_per_chan = tpc;
      a.nslices = c.nslices;
      a.slice_len = c.slice_len;
      a.write_mode = add ? xeng::WM_ADD : xeng::WM_STORE;
      a.head_tiles = (int)c.head;
      a.tail_slices = c.tail_slices;
      a.tail_len = c.tail_len;
      e = xeng::launch_packed(a, s);
      if (e != hipSuccess) return hip_fail(p, e, "packed correlation launch");
    }
  }
  return XENG_OK;
}

// Whether an automatic plan takes such a frame by the packed path (for the
// benchmark's labels; not part of the C ABI in include/xeng.h).
int xeng_takes_packed(int N, int F, int T, int form) {
  return packed_pays(N, F, T, -1, form, false, cu_count_hint());
}

// A plan that serves one call (the Python face's one-shot correlation; not part
// of the C ABI in include/xeng.h): it takes no workspace whose allocation and
// release the one call does not gain back.  Memory from 2 MiB on costs about 35
// us, gigabytes 0.3 ms, less than 2 MiB nothing (one-shot calls, microseconds,
// tiles / workspace): N = 64, F = 4, T = 16384 37 / 63, F = 64, T = 65536
// 165 / 108; N = 128, F = 16, T = 16384 69 / 77; N = 200 (FP8), F = 4, T =
// 16384 53 / 84, F = 16, T = 65536 213 / 168; packed, N = 2048: 3293 / 2729 on
// 1.1e12 complex MACs, 202 / 428 on 1.7e10.
void xeng_plan_once(xeng_plan_t p) { p->once = true; }

static bool once_pays(xeng_plan_t p, size_t bytes, int N, int F, int T, bool packed) {
  if (!p->once || bytes < (2u << 20)) return true;
  if (packed) return 0.5 * N * (N + 1.0) * F * T >= 5e11;
  return tiles_per_channel(N) * F * T >= (1 << 21);
}

// Correlate by the packed path (XENG_ENOMEM: nothing was queued).
static int correlate_packed(xeng_plan_t p, const uint8_t* samples, int N, int F, int T,
                            int32_t* vis, hipStream_t s) {
  const PackedNeed need = packed_need(p, N, F, T);
  if (named_slices(p) > 0 && need.part > kPartMax) return XENG_ENOMEM;
  if (!once_pays(p, need.operands + need.part, N, F, T, true)) return XENG_ENOMEM;
  int rc = workspace(p, need.operands + need.part, s);
  if (rc != XENG_OK) return rc;
  rc = launch_packed_path(p, need, samples, N, F, T, vis, s);
  const int used = workspace_used(p, s);
  if (rc != XENG_OK || used != XENG_OK) return rc != XENG_OK ? rc : used;
  return p->shift ? mark_tables(p, s) : XENG_OK;
}

// Time slices of the channel kernel and the small-array kernel (workgroup
// columns W of a channel, or of the channels that share a small-array
// workgroup).  Microseconds, fitted to frames of 16..256 inputs in 1 to 32
// slices (N = 64, F = 4, T = 8192: 33.9 in one, 13.5 in 8, 11.9 in 32; N = 64,
// F = 256: 34.9 in one, 32.4 in 2, 44.4 in 8): an item takes `tau` per turn (a
// chunk, or the four chunks that the waves of a small workgroup take at once);
// items sharing a CU (up to `occ`) run at 1.7 times the rate of one, at 1.1
// times on whole tile edges (N = 112, F = 46, T = 31552: 66.6 in 5 slices on
// 230 CUs, 86 in 6 that put two on a few CUs, 66.3 in 11 with two on each); the
// frame is read at 4.8 TB/s at best; slices store partial triangles and a second
// launch sums them.
struct Slices {
  int n, len;
};

static Slices channel_slices(xeng_plan_t p, bool small, int N, int F, int len) {
  const int chunks = (len + kChunk - 1) / kChunk;
  const double part = (double)F * N * (N + 1) * sizeof(int32_t);
  const int P = small ? xeng::small_columns(N) : 2 * kTile;
  const int ch = small ? kTile / P : 1, turn = P < kTile ? 4 : 1;
  const double tau = P < 64 ? 0.75 : P == 64 ? 0.96 : P == kTile ? 0.55 : 1.15;
  const int occ = P < 64 ? 3 : P <= kTile ? 2 : 1;
  const long long W = (F + ch - 1) / ch;
  auto slices = [&](int n) {
    const int per = (chunks + n - 1) / n;
    return Slices{(chunks + per - 1) / per, per * kChunk};
  };
  if (p->split_t > 0) return slices(std::min(p->split_t, chunks));
  Slices best = slices(1);
  double cost = 1e300;
  for (int n = 1; n <= std::min(64, (chunks + turn - 1) / turn); ++n) {
    const Slices c = slices(n);
    if (c.n != n) continue;
    if (n > 1 && n * part > 512e6) break;
    const long long items = W * n, slots = (long long)p->cu_count * occ;
    const long long per_cu = (std::min(items, slots) + p->cu_count - 1) / p->cu_count;
    const double item = (c.len / kChunk + turn - 1) / turn * tau *
                        (per_cu > 1 ? per_cu / (P == kTile ? 1.1 : 1.7) : 1.0);
    const double read = (double)F * N * len / 4.8e6;
    const double t = 3.0 + std::max(read, (items + slots - 1) / slots * item) +
                     (n > 1 ? 3.0 + 2.0 * n * part / 2.8e6 : 0.0);
    if (t < cost) {
      cost = t;
      best = c;
    }
  }
  return best;
}

// Estimated microseconds of the channel kernel, as tiles_us; fitted to 700 frames
// of 129..256 inputs, 1..64 channels and 64..65536 samples (9% rms; tiles_us is
// within 16% there).  Short integrations pay for its epilogue (FP8 form, tiles /
// channel kernel: N = 240, F = 56, T = 1843, accumulated 42 / 71; N = 208, F = 8,
// T = 273, accumulated 17 / 28; N = 240, F = 1, T = 205 14 / 19; but N = 256, F =
// 64, T = 32768 297 / 222).
static double channel_us(xeng_plan_t p, int N, int F, int len, bool add) {
  const Slices c = channel_slices(p, false, N, F, len);
  const long long items = (long long)F * c.n;
  const double mb = 4e-6 * F * N * (N + 1.0);
  const double t = 13.4 + 0.875 * ((items + p->cu_count - 1) / p->cu_count) * (c.len / kChunk) +
                   0.293 * mb;
  return c.n > 1 ? t + 2.3 + 0.484 * c.n * mb : add ? t + 7.5 + 0.283 * mb : t;
}

int xeng_correlate(xeng_plan_t p, const uint8_t* samples, int N, int F, int T, int32_t* vis,
                   void* stream) {
  if (!p || !samples || !vis || N < 1 || F < 1 || T < 1) return XENG_EINVAL;
  if (p->kind != PLAN_SINGLE) return XENG_EPLAN;
  if (T > XENG_T_EXACT_MAX) return XENG_EOVERFLOW;
  if (N != p->N || F != p->F || T > p->T_max) return XENG_EPLAN;
  int rc = ensure_cu_count(p);
  if (rc != XENG_OK) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (p->kernel == 0 && packed_pays(N, F, T, p->shift && p->shift_copy ? p->shift_max : -1, p->form,
                                    p->accumulate, p->cu_count) &&
      !stream_captures(s)) {
    rc = correlate_packed(p, samples, N, F, T, vis, s);
    if (rc != XENG_ENOMEM) return rc;
    // no room for the operands: the tile kernels need none
  }
  // delays: in the loads, or by a shifted copy of the frame
  const bool kshift = p->shift && !p->shift_copy;
  if (p->shift && p->shift_copy) {
    hipError_t e = xeng::launch_shift_copy(samples, p->d_shifted, N, F, T, p->d_seg_delay, s);
    if (e != hipSuccess) return hip_fail(p, e, "shift copy launch");
    samples = p->d_shifted;
  }

  const int nt = (N + kTile - 1) / kTile;
  const bool fast = fast_loads(F, N);
  const bool aligned = fast && (N % 16 == 0) && ((reinterpret_cast<uintptr_t>(samples) & 15) == 0);
  // wide tiles (128 x 256, one workgroup per CU) only on request and when
  // the rows allow fast loads; 128 x 128 (two workgroups per CU) otherwise
  const bool wide = aligned && p->kernel == 2 && !kshift;
  // the small-array kernel: automatically up to one tile edge (both forms)
  bool small = p->kernel == 0 && !kshift && N <= kTile;
  // the channel kernel (N <= 256): on request (int8), or automatically above
  // one tile edge; in the FP8 form where it is faster than that form's tiles
  bool chan = !kshift && N <= kChanMax &&
              (p->kernel == 5 ? p->form == XENG_FORM_I8 : p->kernel == 0 && N > kTile && fast);
  if (chan && p->form == XENG_FORM_F8 && p->split_t == 0) {
    const int len = std::min(T, XENG_F8_FLUSH_MAX);
    // (the tiles have to be ahead by a tenth, for the estimates' errors)
    chan = channel_us(p, N, F, len, p->accumulate) <
           1.1 * tiles_us(N, F, len, p->accumulate, p->cu_count);
  }
  int part_slices = 1;  // slices whose partial triangles this call's workspace holds
  if (small || chan) {
    // the slices' partial triangles, as many as the longest launch takes; a call
    // that cannot have them (no memory, or under capture) takes the tile kernels
    part_slices = channel_slices(p, small, N, F, std::min(T, XENG_I8_SEG_MAX)).n;
    if (part_slices > 1) {
      const size_t bytes = (size_t)part_slices * F * N * (N + 1) * sizeof(int32_t);
      // (a plan that names the channel kernel has it)
      const bool most = p->split_t > 0 && p->kernel == 0 && bytes > kPartMax;
      rc = most || stream_captures(s) || !once_pays(p, bytes, N, F, T, false)
               ? XENG_ENOMEM
               : workspace(p, bytes, s);
      if (rc == XENG_ENOMEM) small = chan = false;
      else if (rc != XENG_OK) return rc;
    }
  }
  const long long tpc = wide ? wide_tiles_per_channel(N) : tiles_per_channel(N);
  const int occupancy = wide ? 1 : kOccupancy;
  // The FP8 form integrates at most XENG_F8_FLUSH_MAX samples per launch (f32
  // sums of codes stay exact below 2^24), the int8 form on 128 x 128 tiles at
  // most XENG_I8_SEG_MAX (int32 sums of codes below 2^31); later launches add
  // their sums in stream order.  The wide int8 kernel does the whole frame in
  // one launch.
  const int seg = p->form == XENG_FORM_F8 && !small && !chan ? XENG_F8_FLUSH_MAX
                  : wide                                           ? T
                                                                   : XENG_I8_SEG_MAX;
  for (int t0 = 0; t0 < T; t0 += seg) {
    const int t1 = std::min(T, t0 + seg), len = t1 - t0;
    if (chan || small) {
      // a shorter last segment may want more slices than the first: not more than
      // this call has a workspace for
      const Slices sc = channel_slices(p, small, N, F, len);
      const bool add = p->accumulate || t0 > 0;
      const long long part = (long long)F * N * (N + 1);  // ints of one slice's triangles
      const int ns = std::min(sc.n, part_slices);
      const int sl = ns == sc.n ? sc.len : ((len + ns - 1) / ns + kChunk - 1) / kChunk * kChunk;
      xeng::ChanArgs c;
      c.samples = samples;
      c.vis = vis;
      c.N = N;
      c.F = F;
      c.t0 = t0;
      c.t1 = t1;
      c.nslices = (len + sl - 1) / sl;
      c.slice_len = sl;
      c.row_stride = (long long)F * N;
      c.t_frame = T;
      // one slice writes vis itself; several store their own triangles into
      // the workspace, and a second kernel sums them into vis
      c.partial = ns > 1 ? reinterpret_cast<int32_t*>(p->d_ws) : nullptr;
      c.write_mode = (ns == 1 && add) ? xeng::WM_ADD : xeng::WM_STORE;
      hipError_t e = small ? xeng::launch_small(c, fast, s) : xeng::launch_chan(c, fast, s);
      if (e == hipSuccess && ns > 1)
        e = xeng::launch_chan_reduce(c.partial, vis, part, c.nslices, add, s);
      if (ns > 1) {
        rc = workspace_used(p, s);
        if (rc != XENG_OK) return rc;
      }
      if (e != hipSuccess) return hip_fail(p, e, "channel kernel launch");
      continue;
    }
    const long long W = tpc * F;  // tiles of the launch
    const bool add = p->accumulate || t0 > 0;
    const TileSchedule sch = tile_schedule(W, len, p->cu_count, occupancy, p->split_t, wide);

    xeng::TileArgs a;
    a.samples = samples;
    a.vis = vis;
    a.N = N;
    a.F = F;
    a.t0 = t0;
    a.t1 = t1;
    a.nt = nt;
    a.tiles_per_chan = (int)tpc;
    a.nslices = sch.nslices;
    a.slice_len = sch.slice_len;
    a.row_stride = (long long)F * N;
    a.t_frame = T;
    a.head_tiles = (int)sch.head;
    a.tail_slices = sch.tail_slices;
    a.tail_len = sch.tail_len;
    a.tail_mode = xeng::WM_ATOMIC;
    // Diagonal tiles split the sub-tile above the diagonal between two waves
    // where they are a large share of the tiles (N <= 1024: at least 2 in 9);
    // at N = 2048 (16 in 136) the uniform tile time of the common roles pays
    // more (measured on the full-array frame).
    a.split_diag = p->kernel == 3 ? 1 : p->kernel == 4 ? 0 : (nt <= 8 ? 1 : 0);
    a.seg_delay = kshift ? p->d_seg_delay : nullptr;
    a.blk_delay = kshift ? p->d_blk_delay : nullptr;
    if (sch.nslices > 1) {
      a.write_mode = xeng::WM_ATOMIC;
      if (!add) {
        hipError_t e = xeng::launch_zero(vis, (long long)F * N * (N + 1), s);
        if (e != hipSuccess) return hip_fail(p, e, "zero fill launch");
      }
    } else {
      a.write_mode = add ? xeng::WM_ADD : xeng::WM_STORE;
    }
    if (sch.tail_slices > 0 && !add) {
      hipError_t e = xeng::launch_zero_tiles(vis, N, (int)tpc, nt, (int)sch.head,
                                             (int)(W - sch.head), s);
      if (e != hipSuccess) return hip_fail(p, e, "tail zero launch");
    }
    hipError_t e = wide ? xeng::launch_wide(a, p->form, s) : xeng::launch_tiles(a, p->form, fast, s);
    if (e != hipSuccess) return hip_fail(p, e, "correlation kernel launch");
  }
  return p->shift ? mark_tables(p, s) : XENG_OK;
}

int xeng_correlate_gated(xeng_plan_t p, const uint8_t* samples, int N, int F, int T,
                         const int32_t* gate, int G, int32_t* vis, void* stream) {
  if (!p || !samples || !gate || !vis || N < 1 || F < 1 || T < 1 || G < 1) return XENG_EINVAL;
  if (p->kind != PLAN_SINGLE || p->G_max < 1 || G > p->G_max) return XENG_EPLAN;
  if (T > XENG_T_EXACT_MAX) return XENG_EOVERFLOW;
  if (N != p->N || F != p->F || T > p->T_max) return XENG_EPLAN;
  int rc = ensure_cu_count(p);
  if (rc != XENG_OK) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (p->gate_pending) {
    // the pinned staging may still be read by the previous call's copy
    hipError_t e = hipEventSynchronize(p->gate_done);
    if (e != hipSuccess) return hip_fail(p, e, "hipEventSynchronize");
    p->gate_pending = false;
  }
  // Runs of equal gate per launch segment, grouped by gate in time order,
  // then cut into work gates.  A run is integrated in whole chunks of kChunk
  // samples, and the sums of codes are exact only while a work item
  // integrates at most `seg` chunk-rounded samples.  Runs of 64 samples or
  // more never exceed that (a segment holds at most `seg` samples), but a gate
  // with many shorter runs can: its runs are then split, greedily in time
  // order, into groups that fit, each its own work gate adding into the
  // gate's buffer with int32 atomics (cleared first when the call
  // overwrites).  Two consecutive groups of a gate hold more than `seg`
  // chunk-rounded samples, and a segment holds at most 64 seg of them, so a
  // segment has fewer than kSplitMax extra work gates.
  const int seg = segment_max(p->form);
  const int nseg = (T + seg - 1) / seg;
  long long nruns = 0, ngoff = 0, nvg = 0;
  int* count = p->gate_count.data();
  int* fill = p->gate_fill.data();
  int* zero = p->gate_zero.data();
  std::fill(zero, zero + G, 0);
  for (int k = 0; k < nseg; ++k) {
    const int t0 = k * seg, t1 = std::min(T, t0 + seg);
    const int mode = (p->accumulate || k > 0) ? xeng::WM_ADD : xeng::WM_STORE;
    std::fill(count, count + G, 0);
    for (int t = t0; t < t1;) {  // count the runs of each gate
      const int g = gate[t];
      int u = t + 1;
      while (u < t1 && gate[u] == g) ++u;
      if (g >= 0 && g < G) ++count[g];
      t = u;
    }
    fill[0] = (int)nruns;
    for (int g = 1; g < G; ++g) fill[g] = fill[g - 1] + count[g - 1];
    for (int t = t0; t < t1;) {  // place them, in time order per gate
      const int g = gate[t];
      int u = t + 1;
      while (u < t1 && gate[u] == g) ++u;
      if (g >= 0 && g < G) p->h_runs[fill[g]++] = make_int2(t, u);
      t = u;
    }
    // work gates: fill[g] now ends gate g's runs
    p->seg_goff[k] = (int)ngoff;
    const long long vg0 = nvg;
    int r = (int)nruns;
    for (int g = 0; g < G; ++g) {
      const int r_end = fill[g];
      const long long first = nvg;
      int b = r;
      long long padded = 0;
      for (int e = r; e < r_end; ++e) {
        const int2 run = p->h_runs[e];
        const long long pl = (long long)(run.y - run.x + kChunk - 1) / kChunk * kChunk;
        if (e > b && padded + pl > seg) {
          p->h_gate_off[ngoff++] = b;
          p->h_vgate[nvg++] = make_int2(g, xeng::WM_ATOMIC);
          b = e;
          padded = 0;
        }
        padded += pl;
      }
      const bool split = nvg > first;
      p->h_gate_off[ngoff++] = b;
      p->h_vgate[nvg++] = make_int2(g, split ? xeng::WM_ATOMIC : mode);
      if (split && mode == xeng::WM_STORE) zero[g] = 1;
      r = r_end;
    }
    p->h_gate_off[ngoff++] = r;
    nruns = r;
    p->seg_nvg[k] = (int)(nvg - vg0);
  }
  hipError_t e = hipSuccess;
  if (nruns > 0)
    e = hipMemcpyAsync(p->d_runs, p->h_runs, nruns * sizeof(int2), hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(p->d_gate_off, p->h_gate_off, (size_t)ngoff * sizeof(int),
                       hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(p->d_vgate, p->h_vgate, (size_t)nvg * sizeof(int2), hipMemcpyHostToDevice,
                       s);
  if (e == hipSuccess) e = hipEventRecord(p->gate_done, s);
  if (e != hipSuccess) return hip_fail(p, e, "gate table upload");
  p->gate_pending = true;

  const bool kshift = p->shift && !p->shift_copy;
  if (p->shift && p->shift_copy) {
    e = xeng::launch_shift_copy(samples, p->d_shifted, N, F, T, p->d_seg_delay, s);
    if (e != hipSuccess) return hip_fail(p, e, "shift copy launch");
    samples = p->d_shifted;
  }
  // split gates that overwrite: their buffers are cleared first (the buffers
  // of consecutive gates are contiguous in the gate-major output)
  const long long gate_words = (long long)F * N * (N + 1);
  for (int g = 0; g < G;) {
    if (!zero[g]) {
      ++g;
      continue;
    }
    int h = g;
    while (h < G && zero[h]) ++h;
    e = xeng::launch_zero(vis + g * gate_words, (h - g) * gate_words, s);
    if (e != hipSuccess) return hip_fail(p, e, "gate clear launch");
    g = h;
  }
  for (int k = 0; k < nseg; ++k) {
    xeng::GatedArgs a;
    a.samples = samples;
    a.vis = vis;
    a.N = N;
    a.F = F;
    a.G = p->seg_nvg[k];
    a.nt = (N + kTile - 1) / kTile;
    a.tiles_per_chan = (int)tiles_per_channel(N);
    a.write_mode = (p->accumulate || k > 0) ? xeng::WM_ADD : xeng::WM_STORE;
    a.gate_off = p->d_gate_off + p->seg_goff[k];
    a.runs = p->d_runs;
    a.vgate = p->d_vgate + (p->seg_goff[k] - k);
    a.row_stride = (long long)F * N;
    a.t_frame = T;
    a.seg_delay = kshift ? p->d_seg_delay : nullptr;
    a.blk_delay = kshift ? p->d_blk_delay : nullptr;
    // adding: a work gate without runs adds nothing
    a.skip_empty = a.write_mode == xeng::WM_ADD ? 1 : 0;
    e = xeng::launch_gated(a, p->form, fast_loads(F, N), s);
    if (e != hipSuccess) return hip_fail(p, e, "gated correlation kernel launch");
  }
  return p->shift ? mark_tables(p, s) : XENG_OK;
}

// Event rows a frame of T samples can need per channel: a block of rows never
// takes more event rows than it has rows with several invalid inputs.
static long long flag_rows(int T) { return T; }

int xeng_plan_flagged(xeng_plan_t* out, int N, int F, int T_max, unsigned flags) {
  if (!out) return XENG_EINVAL;
  *out = nullptr;
  xeng_plan_t p = nullptr;
  int rc = xeng_plan(&p, N, F, T_max, flags);
  if (rc != XENG_OK) return rc;
  p->flagged = true;
  p->flag_cap = flag_rows(T_max);
  p->flag_nseg = (int)((p->flag_cap + XENG_I8_SEG_MAX - 1) / XENG_I8_SEG_MAX);
  const long long NB = (long long)N * (N + 1) / 2;
  const long long nint = (long long)F + 2LL * F * N + 1 + 2LL * p->flag_nseg;
  hipError_t e = hipMalloc((void**)&p->d_fU, (size_t)(p->flag_cap * F * N));
  if (e == hipSuccess) e = hipMalloc((void**)&p->d_fX, (size_t)(F * NB * 2) * sizeof(int32_t));
  if (e == hipSuccess) e = hipMalloc((void**)&p->d_fint, (size_t)nint * sizeof(int));
  if (e == hipSuccess) e = hipMalloc((void**)&p->d_fruns, (size_t)p->flag_nseg * sizeof(int2));
  if (e != hipSuccess) {
    rc = e == hipErrorOutOfMemory ? XENG_ENOMEM : XENG_EHIP;
    (void)hipGetLastError();
    xeng_destroy(p);
    return rc;
  }
  *out = p;
  return XENG_OK;
}

int xeng_correlate_flagged(xeng_plan_t p, uint8_t* samples, const uint32_t* flags, int N, int F,
                           int T, int32_t* vis, int32_t* counts, void* stream) {
  if (!p || !samples || !flags || !vis || !counts || N < 1 || F < 1 || T < 1) return XENG_EINVAL;
  if (p->kind != PLAN_SINGLE || !p->flagged || p->shift) return XENG_EPLAN;
  if (T > XENG_T_EXACT_MAX) return XENG_EOVERFLOW;
  if (N != p->N || F != p->F || T > p->T_max) return XENG_EPLAN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  xeng::FlagArgs a;
  a.samples = samples;
  a.flags = flags;
  a.N = N;
  a.F = F;
  a.T = T;
  a.W = (N + 31) / 32;
  a.U = p->d_fU;
  a.cap = flag_rows(T);
  a.cnt = p->d_fint;
  a.single = a.cnt + F;
  a.n = a.single + (long long)F * N;
  a.R = a.n + (long long)F * N;
  a.fgate_off = a.R + 1;
  a.X = p->d_fX;
  a.fruns = p->d_fruns;
  a.counts = counts;
  const int nseg = (int)((a.cap + XENG_I8_SEG_MAX - 1) / XENG_I8_SEG_MAX);
  hipError_t e = xeng::launch_flag_scan(a, nseg, XENG_I8_SEG_MAX, s);
  if (e != hipSuccess) return hip_fail(p, e, "flag scan launch");
  // the frame, now with every flagged sample zero
  int rc = xeng_correlate(p, samples, N, F, T, vis, stream);
  if (rc != XENG_OK) return rc;
  // the event rows: Re X_ij = rows where i and j are both invalid
  for (int k = 0; k < nseg; ++k) {
    xeng::GatedArgs g;
    g.samples = p->d_fU;
    g.vis = p->d_fX;
    g.N = N;
    g.F = F;
    g.G = 1;
    g.nt = (N + kTile - 1) / kTile;
    g.tiles_per_chan = (int)tiles_per_channel(N);
    g.write_mode = k > 0 ? xeng::WM_ADD : xeng::WM_STORE;
    g.gate_off = a.fgate_off + 2 * k;
    g.runs = p->d_fruns;
    g.row_stride = (long long)F * N;
    g.t_frame = (int)p->flag_cap;
    g.seg_delay = nullptr;
    g.blk_delay = nullptr;
    g.vgate = nullptr;
    g.skip_empty = 1;
    e = xeng::launch_gated(g, XENG_FORM_I8, fast_loads(F, N), s);
    if (e != hipSuccess) return hip_fail(p, e, "event correlation kernel launch");
  }
  e = xeng::launch_flag_counts(a, p->accumulate ? 1 : 0, s);
  if (e != hipSuccess) return hip_fail(p, e, "flag count launch");
  return XENG_OK;
}

int xeng_normalize(xeng_plan_t p, const int32_t* vis, const int32_t* counts, double scale,
                   float* out, void* stream) {
  if (!p || !vis || !counts || !out || !(scale > 0.0) || !(scale < 1e300)) return XENG_EINVAL;
  if (p->kind != PLAN_SINGLE) return XENG_EPLAN;
  const long long n = (long long)p->F * p->N * (p->N + 1) / 2;
  hipError_t e = xeng::launch_normalize(vis, counts, n, scale, out,
                                        static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(p, e, "normalize launch");
  return XENG_OK;
}

// Beamforming launches: a launch of T rows reads at byte offsets below
// (T + 512) F N + N + 160 from its first row (more than the rows of one
// workgroup past the frame, plus a step past the row), which the segment
// length keeps below 2^31.
constexpr long long kBeamRowsMax = 512;
long long beam_segment(long long row) { return ((1LL << 31) - 1 - 256) / row - kBeamRowsMax - 2; }

int xeng_plan_beams(xeng_plan_t* out, int N, int F, int T_max, int B, unsigned flags) {
  if (!out) return XENG_EINVAL;
  *out = nullptr;
  if (flags != 0 || B < 1 || B > XENG_BEAMS_MAX) return XENG_EINVAL;
  if (N < 1 || F < 1 || N > XENG_N_MAX || beam_segment((long long)F * N) < 1) return XENG_EINVAL;
  xeng_plan_t p = nullptr;
  int rc = xeng_plan(&p, N, F, T_max, 0);
  if (rc != XENG_OK) return rc;
  p->B = B;
  p->beam_S = (N + 127) / 128;
  p->beam_nbt = (2 * B + 31) / 32;
  const size_t wop_bytes = (size_t)F * p->beam_S * 8 * p->beam_nbt * 64 * 16;
  hipError_t e = hipMalloc(&p->d_wop, wop_bytes);
  if (e == hipSuccess)
    e = hipMalloc((void**)&p->d_bcorr, (size_t)F * p->beam_nbt * 32 * sizeof(int));
  if (e != hipSuccess) {
    rc = e == hipErrorOutOfMemory ? XENG_ENOMEM : XENG_EHIP;
    (void)hipGetLastError();
    xeng_destroy(p);
    return rc;
  }
  *out = p;
  return XENG_OK;
}

int xeng_beam_set_weights(xeng_plan_t p, const int8_t* weights) {
  if (!p || !weights) return XENG_EINVAL;
  if (p->kind != PLAN_SINGLE || p->B < 1) return XENG_EPLAN;
  const int N = p->N, F = p->F, B = p->B, S = p->beam_S, NBT = p->beam_nbt;
  const long long nw = (long long)F * B * N * 2;
  for (long long e = 0; e < nw; ++e)
    if (weights[e] == -128) return XENG_EINVAL;  // -w must be an int8 as well
  // Operand of (f, step s, k-step q, tile c, lane l): bytes e = 0..7 weigh the
  // real code of input 128 s + 32 (q >> 1) + 16 (l >> 5) + 8 (q & 1) + e,
  // bytes 8 + e its imaginary code, for column 32 c + (l & 31) = 2 b + comp of
  // the real contraction: comp 0 (Re y) takes (w_re, -w_im), comp 1 (Im y)
  // (w_im, w_re).
  std::vector<int8_t> wop((size_t)F * S * 8 * NBT * 64 * 16, 0);
  std::vector<int> corr((size_t)F * NBT * 32, 0);
  for (int f = 0; f < F; ++f)
    for (int s = 0; s < S; ++s)
      for (int q = 0; q < 8; ++q)
        for (int c = 0; c < NBT; ++c)
          for (int l = 0; l < 64; ++l) {
            const int col = 32 * c + (l & 31), b = col >> 1, comp = col & 1;
            if (b >= B) continue;
            int8_t* o = &wop[(((((size_t)f * S + s) * 8 + q) * NBT + c) * 64 + l) * 16];
            for (int e = 0; e < 8; ++e) {
              const int n = 128 * s + 32 * (q >> 1) + 16 * (l >> 5) + 8 * (q & 1) + e;
              if (n >= N) continue;
              const int8_t* w = weights + (((size_t)f * B + b) * N + n) * 2;
              const int cr = comp == 0 ? w[0] : w[1];
              const int ci = comp == 0 ? -w[1] : w[0];
              o[e] = (int8_t)cr;
              o[8 + e] = (int8_t)ci;
              corr[(size_t)f * NBT * 32 + col] += 8 * (cr + ci);
            }
          }
  // the plan's last call may still read the old operands
  hipError_t e = wait_tables(p);
  if (e == hipSuccess) e = hipMemcpy(p->d_wop, wop.data(), wop.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(p->d_bcorr, corr.data(), corr.size() * sizeof(int), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(p, e, "beam weight upload");
  p->beams_ready = true;
  return XENG_OK;
}

int xeng_beamform(xeng_plan_t p, const uint8_t* samples, int N, int F, int T, int32_t* beams,
                  void* stream) {
  if (!p || !samples || !beams || N < 1 || F < 1 || T < 1) return XENG_EINVAL;
  if (p->kind != PLAN_SINGLE || p->B < 1 || !p->beams_ready) return XENG_EPLAN;
  if (N != p->N || F != p->F || T > p->T_max) return XENG_EPLAN;
  const int rc = ensure_cu_count(p);
  if (rc != XENG_OK) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const long long row = (long long)F * N;
  const long long seg = beam_segment(row);  // >= 1 by the plan's check
  const bool aligned = (N % 16 == 0) && ((reinterpret_cast<uintptr_t>(samples) & 15) == 0);
  for (long long t0 = 0; t0 < T; t0 += seg) {
    xeng::BeamArgs a;
    a.samples = samples + t0 * row;
    a.beams = beams + t0 * F * 2LL * p->B;
    a.wop = p->d_wop;
    a.corr = p->d_bcorr;
    a.N = N;
    a.F = F;
    a.T = (int)std::min<long long>(seg, T - t0);
    a.B = p->B;
    a.S = p->beam_S;
    a.NBT = p->beam_nbt;
    a.cus = p->cu_count;
    a.tblocks = 0;
    // every launch reads the samples: as few as can be, of about equal tiles
    const int launches = (p->beam_nbt + xeng::kBeamTiles - 1) / xeng::kBeamTiles;
    for (int k = 0, c0 = 0, nb; k < launches; ++k, c0 += nb) {
      nb = (p->beam_nbt - c0 + launches - k - 1) / (launches - k);
      a.c0 = c0;
      const hipError_t e = xeng::launch_beams(a, nb, aligned, s);
      if (e != hipSuccess) return hip_fail(p, e, "beamform kernel launch");
    }
  }
  return mark_tables(p, s);
}

// Estimated microseconds of the batched persistent kernel over `insts`: its work
// items, longest first, on the slots that are free first; stores, atomic adds
// and the clearing before them hide behind long items.  Fitted to 380 batches of 1
// to 48 frames and 900 that packing some of their frames left (10% rms).
static double batch_us(const std::vector<xeng_instance>& insts, int form, bool add, int cus) {
  if (insts.empty()) return 0.0;
  const long long slots = (long long)cus * kOccupancy;
  long long tiles = 0;
  for (const xeng_instance& d : insts) tiles += d.F * tiles_per_channel(d.N);
  const int s_auto = auto_slices(tiles, XENG_T_EXACT_MAX, cus);
  std::vector<std::pair<double, long long>> items;  // samples, how many such items
  double us = 11.9;
  bool cleared = false;
  for (const xeng_instance& d : insts) {
    int S = 0, len = 0;
    batch_slices(d, s_auto, form, S, len);
    items.push_back({(double)std::min(len, d.T), d.F * tiles_per_channel(d.N) * S});
    const double mb = 4e-6 * d.F * d.N * (d.N + 1.0), shown = 500.0 / (500.0 + len);
    us += S > 1 ? (add ? 2.09 : 4.40) * mb * S * shown
                : (0.420 * shown + (add ? 0.174 : 0.118)) * mb;
    cleared |= S > 1 && !add;
  }
  std::sort(items.rbegin(), items.rend());
  typedef std::pair<double, long long> Load;  // samples so far, slots that have them
  std::priority_queue<Load, std::vector<Load>, std::greater<Load>> free;
  free.push({0.0, slots});
  double longest = 0.0, sum = 0.0;
  for (auto [len, n] : items) {
    sum += len * n;
    while (n > 0) {
      const Load l = free.top();
      free.pop();
      const long long k = std::min(n, l.second);
      free.push({l.first + len, k});
      longest = std::max(longest, l.first + len);
      if (l.second > k) free.push({l.first, l.second - k});
      n -= k;
    }
  }
  return us + 0.01045 * longest + 0.0129 * sum / slots + (cleared ? 3.5 : 0.0);
}

// Instances of a batch that run by the packed path, one after another, while
// the persistent kernel takes the others (indices, ascending): the largest
// ones, as many as make the estimated time of the whole call least, if that is
// 5% below the persistent kernel's for all.  In a batch the tiles of all frames
// share the chip, and without its largest frames the others may fill it worse;
// microseconds, persistent kernel for all / by lines in an instance's size alone
// (4 M tile-samples, or 1.1 M where all tiles leave slots unused) / by estimates:
//   16 frames, N 128..2048, F = 4, T <= 8192       407 / 568 / 407
// Of 200 batches of 1 to 48 frames (N 64..2048) 10 are more than 1% slower than
// the persistent kernel alone for it, 2 more than 5%, and their mean is 0.833
// times; by the lines 31, 20 and 0.947.
// A named slice count keeps the tiles.
static std::vector<int> batch_packed_set(const std::vector<xeng_instance>& insts, int form,
                                         bool add, int cus) {
  std::vector<int> large;
  for (int k = 0; k < (int)insts.size(); ++k) {
    const xeng_instance& d = insts[k];
    if (d.split_t == 0 && packed_pays(d.N, d.F, d.T, -1, form, add, cus)) large.push_back(k);
  }
  auto work = [&](int k) { return tiles_per_channel(insts[k].N) * insts[k].F * insts[k].T; };
  std::stable_sort(large.begin(), large.end(), [&](int x, int y) { return work(x) > work(y); });
  double best = 0.95 * batch_us(insts, form, add, cus), packed = 0.0;
  std::vector<char> taken(insts.size(), 0);
  size_t take = 0;
  const size_t step = (large.size() + 31) / 32;  // at most 32 cuts
  for (size_t m = 0; m < large.size() && packed < best; ++m) {
    const xeng_instance& d = insts[large[m]];
    packed += packed_frame_us(d.N, d.F, d.T, add, cus);
    taken[large[m]] = 1;
    if ((m + 1) % step != 0 && m + 1 < large.size()) continue;
    std::vector<xeng_instance> others;
    for (size_t k = 0; k < insts.size(); ++k)
      if (!taken[k]) others.push_back(insts[k]);
    const double t = packed + batch_us(others, form, add, cus);
    if (t < best) {
      best = t;
      take = m + 1;
    }
  }
  large.resize(take);
  std::sort(large.begin(), large.end());
  return large;
}

// pack: some instances may run by the packed path
static int plan_batch(xeng_plan_t* out, const xeng_instance* descs, int count, unsigned flags,
                      bool pack) {
  if (!out) return XENG_EINVAL;
  *out = nullptr;
  if (!descs || count < 1 || !flags_ok(flags, true)) return XENG_EINVAL;
  for (int k = 0; k < count; ++k) {
    const xeng_instance& d = descs[k];
    if (d.N < 1 || d.F < 1 || d.T < 1 || d.N > XENG_N_MAX || d.split_t < 0) return XENG_EINVAL;
  }
  for (int k = 0; k < count; ++k)
    if (descs[k].T > XENG_T_EXACT_MAX) return XENG_EOVERFLOW;
  xeng_plan_t p = new (std::nothrow) xeng_plan_s();
  if (!p) return XENG_ENOMEM;
  p->kind = PLAN_BATCH;
  p->flags = flags;
  p->form = (int)(flags & XENG_FORM_MASK);
  p->accumulate = (flags & XENG_ACCUMULATE) != 0;
  const bool shared = (flags & XENG_SHARED_VIS) != 0;
  try {
    p->insts.assign(descs, descs + count);
    p->inst_zero.assign(count, 0);
    struct Costed {
      long long cost;
      xeng::BatchItem it;
    };
    std::vector<Costed> work;
    // automatic slices (split_t = 0): one count for the whole batch, from its
    // total tiles, so that a launch of few instances still fills the GPU
    long long batch_tiles = 0;
    for (int k = 0; k < count; ++k) batch_tiles += descs[k].F * tiles_per_channel(descs[k].N);
    const int s_auto = auto_slices(batch_tiles, XENG_T_EXACT_MAX, cu_count_hint());
    for (int k = 0; k < count; ++k) {
      const xeng_instance& d = descs[k];
      const int nt = (d.N + kTile - 1) / kTile;
      int S = 0, len = 0;
      batch_slices(d, s_auto, p->form, S, len);
      const int mode = (S > 1 || shared) ? xeng::WM_ATOMIC
                                         : (p->accumulate ? xeng::WM_ADD : xeng::WM_STORE);
      if (S > 1 && !p->accumulate) {
        p->inst_zero[k] = 1;
        p->any_zero = true;
      }
      for (int f = 0; f < d.F; ++f)
        for (int I = 0; I < nt; ++I)
          for (int J = I; J < nt; ++J)
            for (int s = 0; s < S; ++s) {
              xeng::BatchItem it;
              it.inst = k;
              it.f = f;
              it.I = I;
              it.J = J;
              it.t0 = s * len;
              it.t1 = std::min(d.T, (s + 1) * len);
              it.mode = mode;
              it.t_fast = xeng::fast_rows(d.T, d.N, f, d.F);
              // cost: MFMA blocks that hold baselines x samples
              const int rows = std::min(kTile, d.N - I * kTile);
              const int cols = std::min(kTile, d.N - J * kTile);
              long long area = I == J ? (long long)rows * (rows + 1) / 2 : (long long)rows * cols;
              work.push_back({area * (it.t1 - it.t0), it});
            }
    }
    std::stable_sort(work.begin(), work.end(),
                     [](const Costed& x, const Costed& y) { return x.cost > y.cost; });
    p->items.reserve(work.size());
    for (const Costed& c : work) p->items.push_back(c.it);
  } catch (const std::bad_alloc&) {
    delete p;
    return XENG_ENOMEM;
  }
  if (p->items.size() > 0x7fffffffu) {
    delete p;
    return XENG_EINVAL;
  }
  if (pack && !shared) {  // (a vis shared between instances takes atomic adds: tiles)
    try {
      p->large = batch_packed_set(p->insts, p->form, p->accumulate, cu_count_hint());
      std::vector<xeng_instance> others;
      for (int k = 0, l = 0; k < count; ++k) {
        if (l < (int)p->large.size() && p->large[l] == k)
          ++l;
        else
          others.push_back(descs[k]);
      }
      if (!p->large.empty() && !others.empty()) {
        const int rc = plan_batch(&p->rest, others.data(), (int)others.size(), flags, false);
        if (rc != XENG_OK) {
          xeng_destroy(p);
          return rc;
        }
      }
    } catch (const std::bad_alloc&) {
      xeng_destroy(p);
      return XENG_ENOMEM;
    }
  }
  *out = p;
  return XENG_OK;
}

int xeng_plan_batch(xeng_plan_t* out, const xeng_instance* descs, int count, unsigned flags) {
  return plan_batch(out, descs, count, flags, true);
}

static int batch_setup(xeng_plan_t p) {
  if (p->d_items) return XENG_OK;
  int rc = ensure_cu_count(p);
  if (rc != XENG_OK) return rc;
  const size_t ni = p->insts.size(), nw = p->items.size();
  hipError_t e = hipHostMalloc((void**)&p->h_insts, kStageRing * ni * sizeof(xeng::BatchInst),
                               hipHostMallocDefault);
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? XENG_ENOMEM : hip_fail(p, e, "hipHostMalloc");
  e = hipMalloc((void**)&p->d_insts, ni * sizeof(xeng::BatchInst));
  if (e == hipSuccess) e = hipMalloc((void**)&p->d_items, nw * sizeof(xeng::BatchItem));
  if (e == hipSuccess) e = hipMalloc((void**)&p->d_counter, sizeof(int));
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? XENG_ENOMEM : hip_fail(p, e, "hipMalloc");
  e = hipMemcpy(p->d_items, p->items.data(), nw * sizeof(xeng::BatchItem), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(p, e, "work list upload");
  for (int r = 0; r < kStageRing && e == hipSuccess; ++r)
    e = hipEventCreateWithFlags(&p->copy_done[r], hipEventDisableTiming);
  if (e != hipSuccess) return hip_fail(p, e, "hipEventCreate");
  return XENG_OK;
}

// Bring the device instance table up to date with these pointers (a no-op
// when they are the ones already uploaded).
static int batch_upload(xeng_plan_t p, const uint8_t* const* samples, int32_t* const* vis,
                        hipStream_t s) {
  const size_t ni = p->insts.size();
  bool same = p->uploaded.size() == 2 * ni;
  for (size_t k = 0; same && k < ni; ++k)
    same = p->uploaded[2 * k] == samples[k] &&
           p->uploaded[2 * k + 1] == (samples[k] ? vis[k] : nullptr);
  if (same) return XENG_OK;
  const int r = p->stage_next;
  p->stage_next = (r + 1) % kStageRing;
  if (p->copy_pending[r]) {
    // this staging copy may still be read by an earlier call's upload
    hipError_t e = hipEventSynchronize(p->copy_done[r]);
    if (e != hipSuccess) return hip_fail(p, e, "hipEventSynchronize");
    p->copy_pending[r] = false;
  }
  xeng::BatchInst* stage = p->h_insts + (size_t)r * ni;
  p->uploaded.assign(2 * ni, nullptr);
  for (size_t k = 0; k < ni; ++k) {
    const xeng_instance& d = p->insts[k];
    xeng::BatchInst& b = stage[k];
    b.samples = samples[k];
    b.vis = samples[k] ? vis[k] : nullptr;
    b.N = d.N;
    b.F = d.F;
    b.T = d.T;
    b.fast = fast_loads(d.F, d.N);
    b.zero = samples[k] ? p->inst_zero[k] : 0;
    b.pad = 0;
    p->uploaded[2 * k] = samples[k];
    p->uploaded[2 * k + 1] = b.vis;
  }
  hipError_t e = hipMemcpyAsync(p->d_insts, stage, ni * sizeof(xeng::BatchInst),
                                hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipEventRecord(p->copy_done[r], s);
  if (e != hipSuccess) {
    p->uploaded.clear();
    return hip_fail(p, e, "instance table upload");
  }
  p->copy_pending[r] = true;
  return XENG_OK;
}

static int batch_check(xeng_plan_t p, const uint8_t* const* samples, int32_t* const* vis) {
  if (!p || !samples || !vis) return XENG_EINVAL;
  if (p->kind != PLAN_BATCH) return XENG_EPLAN;
  for (size_t k = 0; k < p->insts.size(); ++k)
    if (samples[k] && !vis[k]) return XENG_EINVAL;
  return XENG_OK;
}

static int batch_grid(xeng_plan_t p) {
  const long long g = std::min<long long>((long long)p->cu_count * kOccupancy,
                                          (long long)p->items.size());
  return (int)std::max(1LL, g);
}

// A batch with instances for the packed path: those one by one, the others by
// their own plan.  *done stays false if the call has to take the persistent
// kernel for all: under capture (see stream_captures), or without the memory.
static int batch_packed(xeng_plan_t p, const uint8_t* const* samples, int32_t* const* vis,
                        void* stream, bool graph, bool* done) {
  *done = false;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (p->large.empty() || stream_captures(s)) return XENG_OK;
  int rc = ensure_cu_count(p);
  if (rc != XENG_OK) return rc;
  size_t need = 0;
  for (int k : p->large) {
    if (!samples[k]) continue;
    const xeng_instance& d = p->insts[k];
    const PackedNeed n = packed_need(p, d.N, d.F, d.T);
    need = std::max(need, n.operands + n.part);
  }
  if (need) {
    rc = workspace(p, need, s);
    if (rc != XENG_OK) return rc == XENG_ENOMEM ? XENG_OK : rc;
  }
  if (p->rest) {
    std::vector<const uint8_t*> x;
    std::vector<int32_t*> v;
    try {
      for (size_t k = 0, l = 0; k < p->insts.size(); ++k) {
        if (l < p->large.size() && p->large[l] == (int)k) {
          ++l;
          continue;
        }
        x.push_back(samples[k]);
        v.push_back(vis[k]);
      }
    } catch (const std::bad_alloc&) {
      return XENG_ENOMEM;
    }
    rc = graph ? xeng_correlate_batch_graph(p->rest, x.data(), v.data(), stream)
               : xeng_correlate_batch(p->rest, x.data(), v.data(), stream);
    if (rc != XENG_OK) {
      p->err = p->rest->err;
      return rc;
    }
  }
  for (int k : p->large) {
    if (!samples[k]) continue;
    const xeng_instance& d = p->insts[k];
    rc = correlate_packed(p, samples[k], d.N, d.F, d.T, vis[k], s);
    if (rc != XENG_OK) return rc;
  }
  *done = true;
  return XENG_OK;
}

int xeng_correlate_batch(xeng_plan_t p, const uint8_t* const* samples, int32_t* const* vis,
                         void* stream) {
  int rc = batch_check(p, samples, vis);
  if (rc != XENG_OK) return rc;
  // also before calls by the packed path: a later call under capture takes the
  // persistent kernel for all instances, and can neither allocate its tables nor
  // have its pointers copied from staging that later calls refill
  rc = batch_setup(p);
  if (rc != XENG_OK) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  rc = batch_upload(p, samples, vis, s);
  if (rc != XENG_OK) return rc;
  bool done = false;
  rc = batch_packed(p, samples, vis, stream, false, &done);
  if (rc != XENG_OK || done) return rc;
  hipError_t e = xeng::launch_batch(p->d_insts, (int)p->insts.size(), p->d_items,
                                    (int)p->items.size(), p->d_counter, batch_grid(p), p->form,
                                    p->any_zero, s);
  if (e != hipSuccess) return hip_fail(p, e, "batch kernel launch");
  return XENG_OK;
}

int xeng_correlate_batch_graph(xeng_plan_t p, const uint8_t* const* samples,
                               int32_t* const* vis, void* stream) {
  int rc = batch_check(p, samples, vis);
  if (rc != XENG_OK) return rc;
  // a graph cannot be launched into a capture: its kernels are captured instead
  if (stream_captures(static_cast<hipStream_t>(stream)))
    return xeng_correlate_batch(p, samples, vis, stream);
  rc = batch_setup(p);  // see xeng_correlate_batch
  if (rc != XENG_OK) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  rc = batch_upload(p, samples, vis, s);
  if (rc != XENG_OK) return rc;
  bool done = false;
  rc = batch_packed(p, samples, vis, stream, true, &done);
  if (rc != XENG_OK || done) return rc;
  if (!p->graph_exec) {
    // The kernels read every pointer from the device instance table, so one
    // captured graph serves every set of buffers.
    hipError_t e = hipStreamCreateWithFlags(&p->capture_stream, hipStreamNonBlocking);
    if (e != hipSuccess) return hip_fail(p, e, "hipStreamCreate");
    e = hipStreamBeginCapture(p->capture_stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return hip_fail(p, e, "hipStreamBeginCapture");
    hipError_t le = xeng::launch_batch(p->d_insts, (int)p->insts.size(), p->d_items,
                                       (int)p->items.size(), p->d_counter, batch_grid(p),
                                       p->form, p->any_zero, p->capture_stream);
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(p->capture_stream, &g);
    if (le != hipSuccess) {
      if (g) (void)hipGraphDestroy(g);
      return hip_fail(p, le, "batch kernel capture");
    }
    if (e != hipSuccess) return hip_fail(p, e, "hipStreamEndCapture");
    e = hipGraphInstantiate(&p->graph_exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
      p->graph_exec = nullptr;
      return hip_fail(p, e, "hipGraphInstantiate");
    }
  }
  hipError_t e = hipGraphLaunch(p->graph_exec, s);
  if (e != hipSuccess) return hip_fail(p, e, "hipGraphLaunch");
  return XENG_OK;
}

int xeng_correlate_batch_noalloc(const xeng_instance* descs, int count, unsigned flags,
                                 const uint8_t* const* samples, int32_t* const* vis,
                                 void* stream) {
  if (!descs || !samples || !vis || count < 1 || !flags_ok(flags, true)) return XENG_EINVAL;
  int active = 0;
  for (int k = 0; k < count; ++k) {
    const xeng_instance& d = descs[k];
    if (d.N < 1 || d.F < 1 || d.T < 1 || d.N > XENG_N_MAX || d.split_t < 0) return XENG_EINVAL;
    if (samples[k] && !vis[k]) return XENG_EINVAL;
    active += samples[k] ? 1 : 0;
  }
  for (int k = 0; k < count; ++k)
    if (descs[k].T > XENG_T_EXACT_MAX) return XENG_EOVERFLOW;
  if (active > XENG_NOALLOC_INST_MAX) return XENG_ELIMIT;
  // every tile takes at least one work item
  long long tiles = 0;
  for (int k = 0; k < count; ++k)
    if (samples[k]) tiles += descs[k].F * tiles_per_channel(descs[k].N);
  if (tiles > XENG_NOALLOC_ITEMS_MAX) return XENG_ELIMIT;
  if (active == 0) return XENG_OK;

  unsigned char* ws = nullptr;
  int cus = 0;
  if (xeng::noalloc_workspace(&ws, &cus) != hipSuccess) {
    (void)hipGetLastError();
    return XENG_EHIP;
  }
  const int form = (int)(flags & XENG_FORM_MASK);
  const bool accumulate = (flags & XENG_ACCUMULATE) != 0;
  const bool shared = (flags & XENG_SHARED_VIS) != 0;
  // the same schedule rules as xeng_plan_batch, over the active instances;
  // instances go in decreasing order of their largest work item, so that
  // the longest items start first
  const int s_auto = auto_slices(tiles, XENG_T_EXACT_MAX, cus);
  xeng::NoallocArgs a;
  long long cost[XENG_NOALLOC_INST_MAX];
  int order[XENG_NOALLOC_INST_MAX];
  int n = 0;
  long long nitems = 0;
  bool any_zero = false;
  for (int k = 0; k < count; ++k) {
    if (!samples[k]) continue;
    const xeng_instance& d = descs[k];
    xeng::NoallocInst& in = a.inst[n];
    int S = 0, len = 0;
    batch_slices(d, s_auto, form, S, len);
    const int mode = (S > 1 || shared) ? xeng::WM_ATOMIC
                                       : (accumulate ? xeng::WM_ADD : xeng::WM_STORE);
    const bool zero = S > 1 && !accumulate;
    in.samples = samples[k];
    in.vis = vis[k];
    in.N = d.N;
    in.F = d.F;
    in.T = d.T;
    in.S = S;
    in.len = len;
    in.flags = mode | (zero ? 4 : 0) | (fast_loads(d.F, d.N) ? 8 : 0);
    in.first = 0;
    in.pad = 0;
    any_zero |= zero;
    nitems += (long long)d.F * tiles_per_channel(d.N) * S;
    const long long edge = std::min(kTile, d.N);
    cost[n] = edge * edge * len;
    order[n] = n;
    ++n;
  }
  if (nitems > XENG_NOALLOC_ITEMS_MAX) return XENG_ELIMIT;
  for (int i = 1; i < n; ++i)  // insertion sort by decreasing cost (stable)
    for (int j = i; j > 0 && cost[order[j]] > cost[order[j - 1]]; --j)
      std::swap(order[j], order[j - 1]);
  xeng::NoallocInst sorted[XENG_NOALLOC_INST_MAX];
  int first = 0;
  for (int i = 0; i < n; ++i) {
    sorted[i] = a.inst[order[i]];
    sorted[i].first = first;
    first += sorted[i].F * (int)tiles_per_channel(sorted[i].N) * sorted[i].S;
  }
  std::copy(sorted, sorted + n, a.inst);
  a.ws = ws;
  a.ninst = n;
  a.nitems = (int)nitems;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = xeng::launch_noalloc_prep(a, s);
  if (e == hipSuccess) {
    const int grid = (int)std::max(1LL, std::min<long long>((long long)cus * kOccupancy, nitems));
    e = xeng::launch_batch(reinterpret_cast<const xeng::BatchInst*>(ws + xeng::kNoallocInstOff),
                           n, reinterpret_cast<const xeng::BatchItem*>(ws + xeng::kNoallocItemsOff),
                           (int)nitems, reinterpret_cast<int*>(ws), grid, form, any_zero, s);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return XENG_EHIP;
  }
  return XENG_OK;
}

int xeng_destroy(xeng_plan_t p) {
  if (!p) return XENG_OK;
  if (p->rest) (void)xeng_destroy(p->rest);
  if (p->graph_exec) (void)hipGraphExecDestroy(p->graph_exec);
  if (p->capture_stream) (void)hipStreamDestroy(p->capture_stream);
  for (int r = 0; r < kStageRing; ++r)
    if (p->copy_done[r]) (void)hipEventDestroy(p->copy_done[r]);
  if (p->d_insts) (void)hipFree(p->d_insts);
  if (p->d_items) (void)hipFree(p->d_items);
  if (p->d_counter) (void)hipFree(p->d_counter);
  if (p->h_insts) (void)hipHostFree(p->h_insts);
  if (p->gate_done) (void)hipEventDestroy(p->gate_done);
  if (p->d_gate_off) (void)hipFree(p->d_gate_off);
  if (p->d_runs) (void)hipFree(p->d_runs);
  if (p->h_gate_off) (void)hipHostFree(p->h_gate_off);
  if (p->h_runs) (void)hipHostFree(p->h_runs);
  if (p->d_vgate) (void)hipFree(p->d_vgate);
  if (p->h_vgate) (void)hipHostFree(p->h_vgate);
  if (p->d_seg_delay) (void)hipFree(p->d_seg_delay);
  if (p->d_blk_delay) (void)hipFree(p->d_blk_delay);
  if (p->d_shifted) (void)hipFree(p->d_shifted);
  if (p->d_ws) (void)hipFree(p->d_ws);
  if (p->ws_used) (void)hipEventDestroy(p->ws_used);
  if (p->d_fU) (void)hipFree(p->d_fU);
  if (p->d_fX) (void)hipFree(p->d_fX);
  if (p->d_fint) (void)hipFree(p->d_fint);
  if (p->d_fruns) (void)hipFree(p->d_fruns);
  if (p->d_wop) (void)hipFree(p->d_wop);
  if (p->d_bcorr) (void)hipFree(p->d_bcorr);
  if (p->tables_used) (void)hipEventDestroy(p->tables_used);
  delete p;
  return XENG_OK;
}

}  // extern "C"
