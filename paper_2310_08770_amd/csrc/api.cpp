// Host side of libccpt: argument checking, reference spectra, window tables,
// workspaces, the per-size launch sequence, graph capture and tuning.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <tuple>
#include <vector>

#include "common.h"
#include "tables.h"

using namespace ccpt;

namespace {

bool supported_size(int n) {
  if (n < 16 || n > 512 || (n & 1)) return false;
  int m = n;
  while (m % 2 == 0) m /= 2;
  while (m % 3 == 0) m /= 3;
  return m == 1;
}

// Shape codes.  A square N x N frame has code N.  A rectangle has code
// kRectCode | trans | NY << 11 | NX, NY x NX being its tall kernel shape
// (one of CCPT_FOR_RECT); trans is set when the frame itself is wide (NX rows
// of NY pixels), which the kernels read transposed.  Tables are shared by
// both orientations (key without the trans bit).
constexpr int kRectCode = 1 << 24;
constexpr int kTransBit = 1 << 23;
bool is_rect(int code) { return (code & kRectCode) != 0; }
int code_ny(int code) { return is_rect(code) ? (code >> 11) & 2047 : code; }
int code_nx(int code) { return is_rect(code) ? code & 2047 : code; }
int code_trans(int code) { return is_rect(code) && (code & kTransBit) ? 1 : 0; }
int table_key(int code) { return code & ~kTransBit; }

// The code of an ny x nx frame, 0 if the shape is not supported.
int shape_code(int ny, int nx) {
  if (ny == nx) return supported_size(ny) ? ny : 0;
  const int a = std::max(ny, nx), b = std::min(ny, nx);
  bool ok = false;
#define CASE(p, q) \
  if (a == p && b == q) ok = true;
  CCPT_FOR_RECT(CASE)
#undef CASE
  if (!ok) return 0;
  return kRectCode | (ny < nx ? kTransBit : 0) | (a << 11) | b;
}

struct SizeTables {
  float2* tw = nullptr;  // N
  double2* gy = nullptr;
  double2* gx = nullptr;
  double* gxn = nullptr;
  int ksteps = 0;
  // FP64 mode
  double2* tw64 = nullptr;  // N
};

struct Ref {
  int n = 0;                  // shape code
  float2* spec = nullptr;     // conj F[B], N x (N/2+1) (the adjoint always uses it)
  double2* spec64 = nullptr;  // the same in FP64 (FP64 mode)
  float* img = nullptr;       // E as float (N x N), kept for the CC-SN chain rule
  float2* espec = nullptr;    // CC-SN: F[E], N x (N/2+1), for real-time updates
};

// Launch plan of one frame shape (ccpt_plan): chunk size and block plans.
struct Schedule {
  int chunk = 0;          // frames per launch chunk (0 = default)
  int split_blocks = -1;  // spread a frame over blocks in launches of fewer than this many frames (-1: default)
  int fused_min = -1;     // 256x256: one-kernel correlation from this many frames (-1: default)
};

// Size groups of one call run concurrently on up to kMaxLanes streams.
constexpr int kMaxLanes = 4;

// What decides the launches of a call, and the addresses they hold, beside the
// context's own (whose changes drop the graphs).
struct GraphKey {
  std::vector<int> sig;     // group sizes and counts
  std::vector<char> pairs;  // by group: which correlation its pixels allow
  bool small;               // launches of what fits 192 MB
  const void* out;
  hipStream_t stream;
  bool operator<(const GraphKey& o) const {
    return std::tie(sig, pairs, small, out, stream) < std::tie(o.sig, o.pairs, o.small, o.out, o.stream);
  }
};

}  // namespace

struct ccpt_ctx {
  int device = 0;
  ccpt_options o{};
  int M = 0, c = 0;
  std::map<int, SizeTables> tables;
  // window expansion: half width and the grid's Chebyshev tables
  double half = 0.0;
  float* tf = nullptr;
  double* td = nullptr;
  std::vector<Ref> refs;
  std::map<int, Schedule> sched;
  // workspace
  char* ws = nullptr;
  size_t ws_bytes = 0;
  size_t ws_refused = ~(size_t)0;  // the last workspace that the card had no room for
  size_t ws_room = 0;              // what it had then
  // descriptors
  FrameDesc* d_desc = nullptr;
  FrameDesc* h_desc = nullptr;
  size_t desc_cap = 0;
  std::vector<FrameDesc> last_desc;
  hipEvent_t desc_evt = nullptr;
  // captured graphs
  std::map<GraphKey, hipGraphExec_t> graphs;
  // profiling: events bracketing each launch
  struct Span {
    int stage;
    hipEvent_t a, b;
  };
  std::vector<Span> spans;
  std::vector<hipEvent_t> ev_pool;
  hipStream_t cur_stream = nullptr;
  hipEvent_t open_ev = nullptr;
  // adjoint: packed-gradient offsets + accumulator pointers, accumulators
  void* gsmall = nullptr;
  size_t gsmall_cap = 0;
  char* h_small = nullptr;
  size_t h_small_cap = 0;
  hipEvent_t small_evt = nullptr;
  void* acc_buf = nullptr;
  size_t acc_cap = 0;
  // per-frame states of a chunk: kept in the initial state between chunks by
  // the Newton kernel; re-initialised after a failed launch
  FrameState* st_buf = nullptr;
  size_t st_cap = 0;
  bool st_dirty = true;
  // chunk slots: a group of several chunks runs them alternately on the
  // caller's stream and `aux`, each slot with its own part of the workspace
  // and frame states (CallMem's strides)
  hipStream_t aux = nullptr;
  hipEvent_t fork_evt = nullptr, join_evt = nullptr;
  // concurrent size groups: lane 0 is the caller's stream, lanes 1.. these
  // context-owned streams (default priority), forked from and joined back
  // into the caller's stream by events; each lane has its own workspace and
  // frame states
  hipStream_t lane_s[kMaxLanes - 1] = {};
  hipEvent_t lane_evt[kMaxLanes - 1] = {};
  int lanes = 0;  // most lanes a call uses (0: kMaxLanes)
  // references: check flags, scratch spectrum
  void* ref_flags = nullptr;
  size_t ref_flags_cap = 0;
  void* ref_tmp = nullptr;
  size_t ref_tmp_cap = 0;
  // real-time updates: scratch spectra T and F
  void* rt_buf = nullptr;
  size_t rt_cap = 0;
  // errors
  int last_code = CCPT_OK;
  std::string last_msg;
};

namespace {

int fail(ccpt_ctx* ctx, int code, const char* fmt, ...) __attribute__((format(printf, 3, 4)));
int fail(ccpt_ctx* ctx, int code, const char* fmt, ...) {
  if (ctx) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    ctx->last_code = code;
    ctx->last_msg = buf;
  }
  return code;
}

// A failed call is reported by this library's call that made it: its error is
// taken off the runtime, whose last error the launches read.
#define HIP_CHECK(ctx, call)                                                               \
  do {                                                                                     \
    hipError_t e_ = (call);                                                                \
    if (e_ != hipSuccess) {                                                                \
      (void)hipGetLastError();                                                             \
      return fail(ctx, CCPT_E_HIP, "%s failed: %s", #call, hipGetErrorString(e_));         \
    }                                                                                      \
  } while (0)

// Device and pinned host memory; false (p null, no error left) if refused.
template <typename T>
bool device_alloc(T*& p, size_t bytes) {
  if (hipMalloc((void**)&p, bytes) == hipSuccess) return true;
  (void)hipGetLastError();
  p = nullptr;
  return false;
}
template <typename T>
bool pinned_alloc(T*& p, size_t bytes) {
  if (hipHostMalloc((void**)&p, bytes, hipHostMallocDefault) == hipSuccess) return true;
  (void)hipGetLastError();
  p = nullptr;
  return false;
}

int set_device(ccpt_ctx* ctx) {
  HIP_CHECK(ctx, hipSetDevice(ctx->device));
  return CCPT_OK;
}

bool fp64(const ccpt_ctx* ctx) { return ctx->o.precision == CCPT_PREC_FP64; }

// Longest Newton step before the result falls back to the grid estimate.
// An FP64 grid locates the maximum to a grid step, so a longer step means
// Newton and grid disagree.  FP32 and split-precision grids do not: where
// the correlation is flat near its maximum relative to its size (broad
// spots, the large constant term of CC-SN, large u) neighbouring grid values
// differ by less than their rounding, and the grid maximum can sit tenths of
// a pixel from the true one; their steps are bounded by the half window
// only (the Hessian test and the window test still apply).
double step_limit(const ccpt_ctx* ctx) {
  const double grid = 1.0 / ctx->o.upsample;
  return fp64(ctx) ? grid : std::max(grid, 0.5 * ctx->o.window);
}

// A device copy of src; dst stays null if it fails.
template <typename T>
int upload(ccpt_ctx* ctx, T*& dst, const std::vector<T>& src) {
  T* p = nullptr;
  HIP_CHECK(ctx, hipMalloc(&p, src.size() * sizeof(T)));
  if (hipMemcpy(p, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipFree(p);
    return fail(ctx, CCPT_E_HIP, "copying a table to the device failed");
  }
  dst = p;
  return CCPT_OK;
}

// Frees a reference's buffers and leaves it without a shape.
void free_ref(Ref& r) {
  for (void* p : {(void*)r.spec, (void*)r.spec64, (void*)r.img, (void*)r.espec})
    if (p) (void)hipFree(p);
  r = Ref{};
}

void free_tables(SizeTables& t) {
  for (void* p : {(void*)t.tw, (void*)t.gy, (void*)t.gx, (void*)t.gxn, (void*)t.tw64})
    if (p) (void)hipFree(p);
}

int ensure_tables(ccpt_ctx* ctx, int code) {
  const int key = table_key(code);
  if (ctx->tables.count(key)) return CCPT_OK;
  const int n = code_ny(code), nx = code_nx(code);
  SizeTables t;
  const std::vector<double2> tw = twiddles(n);
  std::vector<float2> tw32(n);
  for (int m = 0; m < n; ++m) tw32[m] = make_float2((float)tw[m].x, (float)tw[m].y);
  const ShapeTables h = build_shape_tables(n, nx, ctx->half);
  t.ksteps = h.ksteps;
  int rc = upload(ctx, t.tw, tw32);
  if (!rc) rc = upload(ctx, t.gy, h.gy);
  if (!rc) rc = upload(ctx, t.gx, h.gx);
  if (!rc) rc = upload(ctx, t.gxn, h.gxn);
  if (!rc && fp64(ctx)) rc = upload(ctx, t.tw64, tw);
  // the grid's tables, once per context: in FP64 in the FP64 mode, else in FP32
  if (!rc && !ctx->tf && !ctx->td) {
    const GridTables g = build_grid_tables(ctx->o.upsample, ctx->M, ctx->c, ctx->half);
    rc = fp64(ctx) ? upload(ctx, ctx->td, g.td) : upload(ctx, ctx->tf, g.tf);
  }
  if (rc) {
    free_tables(t);
    return rc;
  }
  ctx->tables[key] = t;
  return CCPT_OK;
}

// Captured graphs bake in workspace and descriptor addresses: drop them
// whenever either is reallocated.
void drop_graphs(ccpt_ctx* ctx) {
  for (auto& kv : ctx->graphs) (void)hipGraphExecDestroy(kv.second);
  ctx->graphs.clear();
}

// A workspace of at least `bytes`.  CCPT_E_NOMEM (no workspace; not recorded as
// the context's error) if it was not given, `why` the runtime's reason.
int grow_ws(ccpt_ctx* ctx, size_t bytes, hipError_t& why) {
  why = hipSuccess;
  if (bytes <= ctx->ws_bytes) return CCPT_OK;
  drop_graphs(ctx);
  if (ctx->ws) {
    HIP_CHECK(ctx, hipDeviceSynchronize());
    HIP_CHECK(ctx, hipFree(ctx->ws));
    ctx->ws = nullptr;
    ctx->ws_bytes = 0;
  }
  why = hipMalloc(&ctx->ws, bytes);
  if (why != hipSuccess) {
    (void)hipGetLastError();
    ctx->ws = nullptr;
    return CCPT_E_NOMEM;
  }
  ctx->ws_bytes = bytes;
  if (bytes >= ctx->ws_refused) ctx->ws_refused = ~(size_t)0;
  return CCPT_OK;
}

int ensure_ws(ccpt_ctx* ctx, size_t bytes) {
  hipError_t why;
  const int rc = grow_ws(ctx, bytes, why);
  return rc == CCPT_E_NOMEM ? fail(ctx, rc, "workspace of %zu bytes", bytes) : rc;
}

// A workspace that the call can do without: as grow_ws, but one that was refused
// is asked for again only when the card has more room than it had then (asking
// gives up the workspace in hand), and never while the stream is captured.
int ask_ws(ccpt_ctx* ctx, size_t bytes, hipStream_t s) {
  size_t left = 0, total = 0;
  if (bytes > ctx->ws_bytes && bytes >= ctx->ws_refused) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    const bool known = hipStreamIsCapturing(s, &st) == hipSuccess && st == hipStreamCaptureStatusNone &&
                       hipMemGetInfo(&left, &total) == hipSuccess;
    if (!known) (void)hipGetLastError();
    left += ctx->ws_bytes;
    if (!known || left <= ctx->ws_room || left < bytes) return CCPT_E_NOMEM;
  }
  hipError_t why;
  const int rc = grow_ws(ctx, bytes, why);
  if (why == hipErrorOutOfMemory) {
    ctx->ws_refused = bytes;
    if (hipMemGetInfo(&left, &total) != hipSuccess) (void)hipGetLastError();
    ctx->ws_room = left;
  }
  return rc;
}

// Half-spectrum elements of one frame (shape code).
size_t spec_elems(int code) { return (size_t)code_ny(code) * (code_nx(code) / 2 + 1); }

// Workspace of one frame: the row-pass intermediate T, whose memory the window
// coefficients take over once the correlation is done, and the spectrum X.
size_t t_bytes(int n, int precision) {
  const size_t el = precision == CCPT_PREC_FP64 ? sizeof(double2) : sizeof(float2);
  const size_t coef = (size_t)window_tiles(code_nx(n)) * kChebN * kChebN * sizeof(double);
  return (std::max(spec_elems(n) * el, coef) + 15) / 16 * 16;
}

size_t frame_ws_bytes(int n, int precision) {
  if (precision == CCPT_PREC_FP64)
    return t_bytes(n, precision) + spec_elems(n) * sizeof(double2) +
           (size_t)(n / row_block64(n)) * sizeof(PeakCand);
  return t_bytes(n, precision) + spec_elems(n) * sizeof(float2);
}

// Frames whose spectra fill 192 MB.  (The split precisions count a second copy
// of the spectrum, which they no longer keep.)  256 x 256 groups take the
// one-kernel correlation or the three passes by units of this size (launches()),
// and a unit of another size would change which frames' sums run in which order.
int unit_frames(int n, int precision) {
  const size_t budget = (size_t)192 << 20;
  size_t b = 2 * spec_elems(n) * (precision == CCPT_PREC_FP64 ? sizeof(double2) : sizeof(float2));
  if (precision == CCPT_PREC_FP64)
    b += (size_t)(n / row_block64(n)) * sizeof(PeakCand);
  else if (precision != CCPT_PREC_FP32)
    b += (size_t)code_nx(n) * ((code_ny(n) + 31) / 32 * 32) * sizeof(unsigned) +
         (size_t)code_ny(n) * sizeof(float2);
  int c = (int)(budget / b);
  return std::max(1, std::min(c, 4096));
}

// Default frames per launch: three blocks per CU of the kernels that take a
// frame per block, or 192 MB of spectra where that is more (and at most 2 GB).
// Small launches cost more than spectra that outgrow the Infinity Cache: us per
// call, launches that stay inside it -> of up to 768 frames, 2048 frames of 256 x 256
// 907 -> 673 (381 frames are a round and a half of blocks; 512, 1024 and 2048
// a launch take 675, 723 and 694), 512 of 512 x 512 1402 -> 1094 (64, 128 and
// 256 a launch: 1372, 1345, 1193), 512 of 128 x 256 184 -> 141.
int default_chunk(int n, int precision) {
  const size_t cap = ((size_t)2 << 30) / frame_ws_bytes(n, precision);
  return std::max(unit_frames(n, precision), (int)std::min<size_t>(768, cap));
}

// The most frames that a default launch takes (launches()): the chunk that is
// reported where none is set.
int default_most(int n, int precision) {
  const int c = default_chunk(n, precision);
  return c + c / 4;
}

// The chunk that a plan sets, 0 for the default launches.  The reported value of
// the default stands for the default: a plan that is read and written back, or
// kept and restored, changes no launch (chunks of that many frames taken as they
// are would end in other launches, give other frames the one-kernel correlation
// and have no smaller ones to fall back to).
int set_chunk(const ccpt_ctx* ctx, int n) {
  auto it = ctx->sched.find(n);
  const int c = it != ctx->sched.end() ? it->second.chunk : 0;
  return c > 0 && c != default_most(n, ctx->o.precision) ? c : 0;
}

int chunk_for(const ccpt_ctx* ctx, int n) {
  const int c = set_chunk(ctx, n);
  return c > 0 ? c : default_most(n, ctx->o.precision);
}

int split_blocks_for(const ccpt_ctx* ctx, int n) {
  auto it = ctx->sched.find(n);
  if (it != ctx->sched.end() && it->second.split_blocks >= 0) return it->second.split_blocks;
  return kSplitBlocks;
}

// Blocks that share one frame's coefficient pass in a launch of `count`
// frames: one from split_blocks frames on (128 blocks of four waves: half the
// CUs, but nothing to add up afterwards), four down to half that, below it one
// per 16 spectrum columns.  The sums' order follows the number of blocks, so
// it changes only at these two lines.
int window_parts(const ccpt_ctx* ctx, int n, int count) {
  const int sb = split_blocks_for(ctx, n), tiles = window_tiles(code_nx(n));
  if (count >= sb) return 1;
  return count >= sb / 2 ? std::min(tiles, 4) : tiles;
}

int fused_min_for(const ccpt_ctx* ctx, int n) {
  // this precision is defined by the one-kernel correlation, for any launch size
  if (ctx->o.precision == CCPT_PREC_FP16X2) return 1;
  auto it = ctx->sched.find(n);
  if (it != ctx->sched.end() && it->second.fused_min >= 0) return it->second.fused_min;
  return kFusedMinFrames;
}

// One launch of a group: its frames and the 256 x 256 correlation's threshold.
struct Launch {
  int count, fused_min;
};

// The launches of a group of `count` frames of shape code n.  A chunk size that
// the plan sets is taken as it is; so are `limit` frames (> 0: the static
// scratch, or `small`: what fits 192 MB).  Default launches may take a quarter
// more than default_chunk instead of leaving a small one for the end.  Frames of
// 256 x 256 take the correlation that they take in units of unit_frames: the
// one-kernel one, but for a last unit below fused_min.
std::vector<Launch> launches(const ccpt_ctx* ctx, int n, int count, bool small, int limit) {
  std::vector<Launch> v;
  const int fm = fused_min_for(ctx, n);
  const int set = set_chunk(ctx, n);
  const int unit = set > 0 ? set : unit_frames(n, ctx->o.precision);
  if (set > 0 || small || limit > 0) {
    const int c = limit > 0 ? std::min(unit, limit) : unit;
    for (int left = count; left > 0 && c > 0; left -= c) v.push_back(Launch{std::min(c, left), fm});
    return v;
  }
  const int chunk = default_chunk(n, ctx->o.precision);
  auto split = [&](int left, int f) {
    while (left > 0) {
      const int c = left <= default_most(n, ctx->o.precision) ? left : chunk;
      v.push_back(Launch{c, f});
      left -= c;
    }
  };
  if (code_ny(n) != 256 || code_nx(n) != 256) {
    split(count, fm);
    return v;
  }
  int fused = 0;  // frames of the units that reach fused_min
  if (std::min(unit, count) >= fm) fused = count % unit >= fm ? count : count - count % unit;
  split(fused, 1);
  split(count - fused, 1 << 30);
  return v;
}

int largest(const std::vector<Launch>& v) {
  int m = 0;
  for (const Launch& l : v) m = std::max(m, l.count);
  return m;
}

// Device memory the launches of one call work in: the context's buffers
// (ccpt_track_batch) or the library's static scratch (ccpt_track_batch_static).
struct CallMem {
  char* ws = nullptr;          // chunk workspace, slot_ws bytes per slot
  size_t slot_ws = 0;
  FrameState* st = nullptr;    // frame states, slot_st entries per slot
  size_t slot_st = 0;
  size_t chunk_bytes = 0;      // > 0: chunks limited to this much workspace
  bool small = false;          // launches of what fits 192 MB
  bool slots = true;           // two chunk slots allowed (CCPT_FLAG_STREAMS)
  bool mark = true;            // profiling events allowed
  bool* st_dirty = nullptr;    // set while a chunk's states may be left non-initial
};

CallMem ctx_mem(ccpt_ctx* ctx) {
  CallMem m;
  m.ws = ctx->ws;
  m.st = ctx->st_buf;
  m.st_dirty = &ctx->st_dirty;
  return m;
}

// Carves the workspace for a chunk of `chunk` frames of size n (every part
// 16-byte aligned: spectra rows hold an even number of float2).
void carve(ccpt_ctx* ctx, const CallMem& mem, int n, int chunk, int slot, GroupParams& g) {
  const size_t spec = spec_elems(n);
  char* ws = mem.ws + slot * mem.slot_ws;
  char* x = ws + t_bytes(n, ctx->o.precision) * chunk;
  g.st = mem.st + slot * mem.slot_st;
  g.coef = (double*)ws;
  g.T = g.X = nullptr;
  g.T64 = g.X64 = nullptr;
  g.cand = nullptr;
  if (fp64(ctx)) {
    g.T64 = (double2*)ws;
    g.X64 = (double2*)x;
    g.cand = (PeakCand*)(g.X64 + spec * chunk);
    g.ncand = n / row_block64(n);
    return;
  }
  g.T = (float2*)ws;
  g.X = (float2*)x;
}

int check_image(ccpt_ctx* ctx, const void* data, int ny, int nx, int pitch, int dtype,
                const char* what, int idx) {
  if (!data) return fail(ctx, CCPT_E_INVALID, "%s %d: null data", what, idx);
  if (dtype != CCPT_U16 && dtype != CCPT_F32 && dtype != CCPT_F64)
    return fail(ctx, CCPT_E_INVALID, "%s %d: unknown dtype %d", what, idx, dtype);
  if (ny <= 0 || nx <= 0 || pitch < nx)
    return fail(ctx, CCPT_E_INVALID, "%s %d: bad shape %dx%d pitch %d", what, idx, ny, nx, pitch);
  if (!shape_code(ny, nx))
    return fail(ctx, CCPT_E_UNSUPPORTED, "%s %d: %dx%d is not a supported shape", what, idx, ny,
                nx);
  const size_t align = dtype_bytes(dtype);
  if ((uintptr_t)data % align)
    return fail(ctx, CCPT_E_INVALID, "%s %d: misaligned data", what, idx);
  return CCPT_OK;
}

// One pixel of a host copy of an image.
double pixel(const void* raw, int dtype, size_t k) {
  if (dtype == CCPT_U16) return (double)((const uint16_t*)raw)[k];
  if (dtype == CCPT_F64) return ((const double*)raw)[k];
  return (double)((const float*)raw)[k];
}

// Calls that work on square frames only (the adjoint, the Fisher information
// and the offline reference).
int require_square(ccpt_ctx* ctx, int ny, int nx, const char* what) {
  if (ny != nx)
    return fail(ctx, CCPT_E_UNSUPPORTED, "%s: %dx%d frames are tracked, but this call takes square "
                "frames only", what, ny, nx);
  return CCPT_OK;
}

GroupParams base_params(ccpt_ctx* ctx, int n) {
  GroupParams g{};
  g.tw = ctx->tables[table_key(n)].tw;
  g.mode = ctx->o.mode;
  g.eps = (float)ctx->o.eps;
  g.eps64 = ctx->o.eps;
  g.tw64 = ctx->tables[table_key(n)].tw64;
  g.trans = code_trans(n);
  g.u = ctx->o.upsample;
  g.M = ctx->M;
  g.c = ctx->c;
  g.newton_iters = ctx->o.newton_iters;
  g.half_window = 0.5 * ctx->o.window;
  g.fused_min = fused_min_for(ctx, n);
  return g;
}

hipEvent_t pool_event(ccpt_ctx* ctx) {
  if (!ctx->ev_pool.empty()) {
    hipEvent_t e = ctx->ev_pool.back();
    ctx->ev_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

void mark_cb(void* user, int stage, int begin) {
  ccpt_ctx* ctx = (ccpt_ctx*)user;
  hipEvent_t e = pool_event(ctx);
  if (!e) return;
  (void)hipEventRecord(e, ctx->cur_stream);
  if (begin) {
    ctx->open_ev = e;
  } else if (ctx->open_ev) {
    ctx->spans.push_back({stage, ctx->open_ev, e});
    ctx->open_ev = nullptr;
  }
}

Marker marker_of(ccpt_ctx* ctx, hipStream_t s) {
  Marker m;
  if (ctx->o.flags & CCPT_FLAG_PROFILE) {
    ctx->cur_stream = s;
    m.fn = mark_cb;
    m.user = ctx;
  }
  return m;
}

// With CCPT_FLAG_STREAMS the chunks of one group run on two streams (not
// when launches are being timed, which needs them in sequence).
bool use_slots(const ccpt_ctx* ctx) {
  return ctx->aux != nullptr && (ctx->o.flags & CCPT_FLAG_STREAMS) &&
         !(ctx->o.flags & CCPT_FLAG_PROFILE);
}

// Frames first..first+count-1 of a plan are uint16 or float32 with an even
// pitch and pixel pairs aligned to their size.
bool pairs_ok(const std::vector<FrameDesc>& desc, int first, int count) {
  for (int i = first; i < first + count; ++i) {
    const FrameDesc& d = desc[i];
    if ((d.dtype != CCPT_U16 && d.dtype != CCPT_F32) || (d.pitch & 1) ||
        ((uintptr_t)d.data & (uintptr_t)(2 * dtype_bytes(d.dtype) - 1)))
      return false;
  }
  return true;
}

// Launches the whole tracking sequence for one size group, chunk by chunk.
int run_group(ccpt_ctx* ctx, const CallMem& mem, int n, const FrameDesc* d_desc, int first,
              int count, ccpt_result* out, hipStream_t s, bool pairs) {
  int limit = 0;
  if (mem.chunk_bytes) {
    limit = std::min<int>((int)(mem.chunk_bytes / frame_ws_bytes(n, ctx->o.precision)), (int)mem.slot_st);
    if (limit < 1) return fail(ctx, CCPT_E_INVALID, "no workspace for one frame");
  }
  const std::vector<Launch> ls = launches(ctx, n, count, mem.small, limit);
  const int chunk = largest(ls);
  SizeTables& t = ctx->tables[table_key(n)];
  const int ny = code_ny(n), nx = code_nx(n);
  const WindowTables wt{t.gy, t.gx, t.gxn, ctx->tf, ctx->td, t.ksteps, ctx->half};
  const Marker mark = mem.mark ? marker_of(ctx, s) : Marker{};
  // several chunks: alternate between the two slots (streams s and aux),
  // forked from and joined back into s
  const bool two = ls.size() > 1 && mem.slots && use_slots(ctx);
  if (two) {
    HIP_CHECK(ctx, hipEventRecord(ctx->fork_evt, s));
    HIP_CHECK(ctx, hipStreamWaitEvent(ctx->aux, ctx->fork_evt, 0));
  }
  // a failed launch leaves no work of this call running on the second stream
  auto failed = [&](const char* what) {
    if (two) (void)hipStreamSynchronize(ctx->aux);
    return fail(ctx, CCPT_E_HIP, "%s launch failed", what);
  };
  int c0 = 0;
  for (size_t ci = 0; ci < ls.size(); c0 += ls[ci++].count) {
    const int slot = two ? (int)(ci & 1) : 0;
    hipStream_t cs = slot ? ctx->aux : s;
    GroupParams g = base_params(ctx, n);
    g.pairs_ok = pairs ? 1 : 0;
    g.desc = d_desc;
    g.first = first + c0;
    g.count = ls[ci].count;
    g.fused_min = ls[ci].fused_min;
    g.out = out;
    carve(ctx, mem, n, chunk, slot, g);
    const int parts = window_parts(ctx, n, g.count);
    if (mem.st_dirty) *mem.st_dirty = true;  // until this chunk's Newton launch has gone in
    if ((fp64(ctx) ? launch_xcorr64(n, g, cs, mark) : launch_xcorr(ny, nx, g, cs, mark)))
      return failed("correlation");
    mark(CCPT_STAGE_UPDFT, 1);
    if (launch_window_coef(ny, nx, g, wt, parts, cs)) return failed("window coefficient");
    mark(CCPT_STAGE_UPDFT, 0);
    mark(CCPT_STAGE_NEWTON, 1);
    if (launch_window_max(ny, nx, g, wt, parts, step_limit(ctx), cs)) return failed("window maximum");
    mark(CCPT_STAGE_NEWTON, 0);
    if (mem.st_dirty) *mem.st_dirty = false;
  }
  if (two) {
    HIP_CHECK(ctx, hipEventRecord(ctx->join_evt, ctx->aux));
    HIP_CHECK(ctx, hipStreamWaitEvent(s, ctx->join_evt, 0));
  }
  return CCPT_OK;
}

// Validated, size-grouped descriptors of a roi array.
struct Plan {
  std::vector<FrameDesc> desc;  // grouped by shape, largest first
  std::vector<int> sig;         // (shape code, count) pairs of the groups
};

// fp32_spec: point the descriptors at the FP32 reference spectra whatever
// the precision (the adjoint works in FP32).
int plan_rois(ccpt_ctx* ctx, const ccpt_roi* rois, int n, Plan& plan, bool fp32_spec = false) {
  if (ctx->refs.empty()) return fail(ctx, CCPT_E_NOREF, "no reference set");
  std::vector<int> code(n);
  for (int i = 0; i < n; ++i) {
    const ccpt_roi& r = rois[i];
    int rc = check_image(ctx, r.data, r.ny, r.nx, r.pitch, r.dtype, "roi", i);
    if (rc) return rc;
    if (r.ref_id < 0 || r.ref_id >= (int)ctx->refs.size())
      return fail(ctx, CCPT_E_NOREF, "roi %d: reference id %d not set", i, r.ref_id);
    code[i] = shape_code(r.ny, r.nx);
    if (ctx->refs[r.ref_id].n != code[i])
      return fail(ctx, CCPT_E_INVALID, "roi %d: shape %dx%d differs from reference %d", i, r.ny,
                  r.nx, r.ref_id);
  }
  // group by shape, largest first (they take longest); stable within a shape
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
    const long pa = (long)rois[a].ny * rois[a].nx, pb = (long)rois[b].ny * rois[b].nx;
    return pa != pb ? pa > pb : code[a] > code[b];
  });
  plan.desc.resize(n);
  plan.sig.clear();
  for (int k = 0; k < n; ++k) {
    const ccpt_roi& r = rois[order[k]];
    FrameDesc d;
    d.data = r.data;
    const Ref& ref = ctx->refs[r.ref_id];
    d.rspec = (fp64(ctx) && !fp32_spec) ? (const void*)ref.spec64 : (const void*)ref.spec;
    d.pitch = r.pitch;
    d.dtype = r.dtype;
    d.out_idx = order[k];
    d.ref_id = r.ref_id;
    plan.desc[k] = d;
    if (plan.sig.empty() || plan.sig[plan.sig.size() - 2] != code[order[k]]) {
      plan.sig.push_back(code[order[k]]);
      plan.sig.push_back(0);
    }
    plan.sig.back()++;
  }
  // FP16X2 runs the one-kernel correlation only, which reads pixel pairs
  if (ctx->o.precision == CCPT_PREC_FP16X2 && !fp32_spec && !pairs_ok(plan.desc, 0, n))
    return fail(ctx, CCPT_E_UNSUPPORTED,
                "the fp16 split takes uint16 or float32 frames with an even pitch and aligned pairs");
  return CCPT_OK;
}

// Copies the descriptors to the context's device table through a pinned
// staging buffer; skipped when identical to the previous upload.
int upload_desc(ccpt_ctx* ctx, const std::vector<FrameDesc>& desc, hipStream_t s) {
  const size_t n = desc.size();
  const size_t bytes = n * sizeof(FrameDesc);
  if (n > ctx->desc_cap) {
    HIP_CHECK(ctx, hipDeviceSynchronize());
    drop_graphs(ctx);
    if (ctx->d_desc) (void)hipFree(ctx->d_desc);
    if (ctx->h_desc) (void)hipHostFree(ctx->h_desc);
    ctx->d_desc = nullptr;
    ctx->h_desc = nullptr;
    size_t cap = std::max<size_t>(n, 64);
    if (!device_alloc(ctx->d_desc, cap * sizeof(FrameDesc)) || !pinned_alloc(ctx->h_desc, cap * sizeof(FrameDesc))) {
      ctx->desc_cap = 0;
      return fail(ctx, CCPT_E_NOMEM, "descriptor table");
    }
    ctx->desc_cap = cap;
    ctx->last_desc.clear();
  }
  const bool same = ctx->last_desc.size() == n &&
                    memcmp(ctx->last_desc.data(), desc.data(), bytes) == 0;
  if (!same) {
    HIP_CHECK(ctx, hipEventSynchronize(ctx->desc_evt));
    memcpy(ctx->h_desc, desc.data(), bytes);
    HIP_CHECK(ctx, hipMemcpyAsync(ctx->d_desc, ctx->h_desc, bytes, hipMemcpyHostToDevice, s));
    HIP_CHECK(ctx, hipEventRecord(ctx->desc_evt, s));
    ctx->last_desc = desc;
  }
  return CCPT_OK;
}

// Device buffer owned by the context, grown on demand.
int ensure_buf(ccpt_ctx* ctx, void*& p, size_t& cap, size_t bytes) {
  if (bytes <= cap) return CCPT_OK;
  if (p) {
    HIP_CHECK(ctx, hipDeviceSynchronize());
    (void)hipFree(p);
    p = nullptr;
    cap = 0;
  }
  if (!device_alloc(p, bytes)) return fail(ctx, CCPT_E_NOMEM, "buffer of %zu bytes", bytes);
  cap = bytes;
  return CCPT_OK;
}

// The frame-state buffer for chunks of up to `count` frames, in the initial
// state (a new buffer, or one left dirty by a failed launch, is initialised on
// stream s before any kernel of the call uses it).
int ensure_state(ccpt_ctx* ctx, size_t count, hipStream_t s) {
  if (count > ctx->st_cap) {
    drop_graphs(ctx);
    size_t cap = ctx->st_cap;
    void* p = ctx->st_buf;
    int rc = ensure_buf(ctx, p, cap, count * sizeof(FrameState));
    ctx->st_buf = (FrameState*)p;
    ctx->st_cap = cap / sizeof(FrameState);
    if (rc) return rc;
    ctx->st_dirty = true;
  }
  if (ctx->st_dirty) {
    if (launch_init_state(ctx->st_buf, (int)ctx->st_cap, s))
      return fail(ctx, CCPT_E_HIP, "state initialisation launch failed");
    ctx->st_dirty = false;
  }
  return CCPT_OK;
}

// The streams and events of lanes 1.. (default priority).
int create_lanes(ccpt_ctx* ctx) {
  for (int l = 0; l < kMaxLanes - 1; ++l)
    if (hipStreamCreateWithFlags(&ctx->lane_s[l], hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&ctx->lane_evt[l], hipEventDisableTiming) != hipSuccess)
      return -1;
  return 0;
}

}  // namespace

// ===================================================================== ABI

extern "C" {

void ccpt_default_options(ccpt_options* o) {
  if (!o) return;
  o->mode = CCPT_MODE_CCU;
  o->eps = 200.0;
  o->upsample = 100;
  o->window = 1.5;
  o->precision = CCPT_PREC_FP32;
  o->newton_iters = 3;
  o->flags = 0;
}

const char* ccpt_status_string(int code) {
  switch (code) {
    case CCPT_OK: return "ok";
    case CCPT_E_INVALID: return "invalid argument";
    case CCPT_E_UNSUPPORTED: return "unsupported frame size";
    case CCPT_E_NOREF: return "no reference for this id";
    case CCPT_E_HIP: return "HIP runtime error";
    case CCPT_E_NONPOSITIVE_REF: return "CC-SN reference has E + eps <= 0";
    case CCPT_E_NOMEM: return "out of memory";
  }
  return "unknown status";
}

int ccpt_last_error(const ccpt_ctx* ctx, char* buf, size_t len) {
  if (!ctx) return CCPT_E_INVALID;
  if (buf && len) {
    size_t k = std::min(len - 1, ctx->last_msg.size());
    memcpy(buf, ctx->last_msg.data(), k);
    buf[k] = 0;
  }
  return ctx->last_code;
}

int ccpt_create(ccpt_ctx** out, int device, const ccpt_options* opts) {
  if (!out) return CCPT_E_INVALID;
  *out = nullptr;
  ccpt_options o;
  if (opts)
    o = *opts;
  else
    ccpt_default_options(&o);
  if (o.mode != CCPT_MODE_CCU && o.mode != CCPT_MODE_CCSN) return CCPT_E_INVALID;
  if (o.upsample < 1 || o.upsample > 1024) return CCPT_E_INVALID;
  if (!(o.window > 0.0 && o.window <= 2.0)) return CCPT_E_INVALID;
  if (o.precision != CCPT_PREC_FP32 && o.precision != CCPT_PREC_BF16X2 &&
      o.precision != CCPT_PREC_FP16X2 &&
      o.precision != CCPT_PREC_FP64)
    return CCPT_E_INVALID;
  if (o.newton_iters < 0 || o.newton_iters > 8) return CCPT_E_INVALID;
  if (!std::isfinite(o.eps)) return CCPT_E_INVALID;
  const int M = (int)std::ceil(o.window * o.upsample - 1e-9);
  if (M < 1 || M > 1536) return CCPT_E_INVALID;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return CCPT_E_HIP;
  ccpt_ctx* ctx = new (std::nothrow) ccpt_ctx();
  if (!ctx) return CCPT_E_NOMEM;
  ctx->device = device;
  ctx->o = o;
  ctx->M = M;
  ctx->c = M / 2;
  ctx->half = window_half(0.5 * o.window, o.upsample, M, ctx->c);
  if (hipSetDevice(device) != hipSuccess || scratch_setup(device) != 0 ||
      hipEventCreateWithFlags(&ctx->desc_evt, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&ctx->fork_evt, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&ctx->join_evt, hipEventDisableTiming) != hipSuccess ||
      hipStreamCreateWithFlags(&ctx->aux, hipStreamNonBlocking) != hipSuccess ||
      create_lanes(ctx) != 0 ||
      hipEventCreateWithFlags(&ctx->small_evt, hipEventDisableTiming) != hipSuccess) {
    ccpt_destroy(ctx);
    return CCPT_E_HIP;
  }
  *out = ctx;
  return CCPT_OK;
}

void ccpt_destroy(ccpt_ctx* ctx) {
  if (!ctx) return;
  (void)hipSetDevice(ctx->device);
  (void)hipDeviceSynchronize();
  for (auto& kv : ctx->graphs) (void)hipGraphExecDestroy(kv.second);
  for (auto& sp : ctx->spans) {
    (void)hipEventDestroy(sp.a);
    (void)hipEventDestroy(sp.b);
  }
  for (auto e : ctx->ev_pool) (void)hipEventDestroy(e);
  for (auto& kv : ctx->tables) free_tables(kv.second);
  if (ctx->tf) (void)hipFree(ctx->tf);
  if (ctx->td) (void)hipFree(ctx->td);
  for (auto& r : ctx->refs) free_ref(r);
  if (ctx->ref_flags) (void)hipFree(ctx->ref_flags);
  if (ctx->ref_tmp) (void)hipFree(ctx->ref_tmp);
  if (ctx->ws) (void)hipFree(ctx->ws);
  if (ctx->d_desc) (void)hipFree(ctx->d_desc);
  if (ctx->h_desc) (void)hipHostFree(ctx->h_desc);
  if (ctx->desc_evt) (void)hipEventDestroy(ctx->desc_evt);
  if (ctx->fork_evt) (void)hipEventDestroy(ctx->fork_evt);
  if (ctx->join_evt) (void)hipEventDestroy(ctx->join_evt);
  if (ctx->aux) (void)hipStreamDestroy(ctx->aux);
  for (int l = 0; l < kMaxLanes - 1; ++l) {
    if (ctx->lane_s[l]) (void)hipStreamDestroy(ctx->lane_s[l]);
    if (ctx->lane_evt[l]) (void)hipEventDestroy(ctx->lane_evt[l]);
  }
  if (ctx->small_evt) (void)hipEventDestroy(ctx->small_evt);
  if (ctx->gsmall) (void)hipFree(ctx->gsmall);
  if (ctx->acc_buf) (void)hipFree(ctx->acc_buf);
  if (ctx->st_buf) (void)hipFree(ctx->st_buf);
  if (ctx->rt_buf) (void)hipFree(ctx->rt_buf);
  if (ctx->h_small) (void)hipHostFree(ctx->h_small);
  delete ctx;
}

int ccpt_set_reference(ccpt_ctx* ctx, const ccpt_image* refs, int n_refs, void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (!refs || n_refs <= 0) return fail(ctx, CCPT_E_INVALID, "no references given");
  int rc = set_device(ctx);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  for (int i = 0; i < n_refs; ++i) {
    rc = check_image(ctx, refs[i].data, refs[i].ny, refs[i].nx, refs[i].pitch, refs[i].dtype,
                     "reference", i);
    if (rc) return rc;
    if (fp64(ctx) && refs[i].ny != refs[i].nx)
      return fail(ctx, CCPT_E_UNSUPPORTED, "reference %d: the FP64 mode takes square frames only",
                  i);
    if (ctx->o.precision == CCPT_PREC_FP16X2 && !(refs[i].ny == 256 && refs[i].nx == 256))
      return fail(ctx, CCPT_E_UNSUPPORTED, "reference %d: the fp16 split takes 256x256 frames only",
                  i);
  }
  // everything queued is done with the old set, and whatever made the images,
  // on any stream, has run
  HIP_CHECK(ctx, hipDeviceSynchronize());
  // the domain checks, on the device: one flag per reference
  rc = ensure_buf(ctx, ctx->ref_flags, ctx->ref_flags_cap, (size_t)n_refs * sizeof(unsigned));
  if (rc) return rc;
  unsigned* flags = (unsigned*)ctx->ref_flags;
  if (launch_zero(flags, (size_t)n_refs * sizeof(unsigned), s))
    return fail(ctx, CCPT_E_HIP, "zero launch failed");
  for (int i = 0; i < n_refs; ++i)
    if (launch_ref_check(refs[i].data, refs[i].dtype, refs[i].pitch, refs[i].ny, refs[i].nx, ctx->o.mode,
                         ctx->o.eps, flags + i, s))
      return fail(ctx, CCPT_E_HIP, "reference check launch failed");
  std::vector<unsigned> bad(n_refs);
  HIP_CHECK(ctx, hipMemcpyAsync(bad.data(), flags, (size_t)n_refs * sizeof(unsigned),
                                hipMemcpyDeviceToHost, s));
  HIP_CHECK(ctx, hipStreamSynchronize(s));
  for (int i = 0; i < n_refs; ++i) {
    if (!bad[i]) continue;
    // the first offending pixel, for the message
    const ccpt_image& im = refs[i];
    std::vector<char> raw(((size_t)(im.ny - 1) * im.pitch + im.nx) * dtype_bytes(im.dtype));
    HIP_CHECK(ctx, hipMemcpy(raw.data(), im.data, raw.size(), hipMemcpyDeviceToHost));
    for (int y = 0; y < im.ny; ++y)
      for (int x = 0; x < im.nx; ++x) {
        const double v = pixel(raw.data(), im.dtype, (size_t)y * im.pitch + x);
        if (!std::isfinite(v))
          return fail(ctx, CCPT_E_INVALID, "reference %d has a non-finite pixel", i);
        if (ctx->o.mode == CCPT_MODE_CCSN && !(v + ctx->o.eps > 0.0))
          return fail(ctx, CCPT_E_NONPOSITIVE_REF, "reference %d: E + eps <= 0 at (%d, %d)", i,
                      y, x);
      }
    return fail(ctx, CCPT_E_INVALID, "reference %d changed while it was read", i);
  }
  ctx->last_desc.clear();
  // scratch: one spectrum (FP64 size)
  size_t tmp_need = 0;
  for (int i = 0; i < n_refs; ++i) {
    const int code = shape_code(refs[i].ny, refs[i].nx);
    tmp_need = std::max(tmp_need, spec_elems(code) * sizeof(double2));
    rc = ensure_tables(ctx, code);
    if (rc) return rc;
  }
  rc = ensure_buf(ctx, ctx->ref_tmp, ctx->ref_tmp_cap, tmp_need);
  if (rc) return rc;
  float2* T = (float2*)ctx->ref_tmp;
  double2* T64 = (double2*)ctx->ref_tmp;
  // a reference of the same shape takes over its predecessor's buffers; after a
  // failure there are no references: some of the new set among what a caller
  // takes for the old one would have other sizes than its gradient arrays
  auto drop_from = [&](size_t k) {
    for (size_t r = k; r < ctx->refs.size(); ++r) free_ref(ctx->refs[r]);
    ctx->refs.resize(std::min(k, ctx->refs.size()));
  };
  auto lost = [&](int code, const char* what) {
    if (hipStreamSynchronize(s) != hipSuccess) (void)hipGetLastError();
    drop_from(0);
    return fail(ctx, code, "%s", what);
  };
  drop_from(n_refs);
  const int weight = ctx->o.mode == CCPT_MODE_CCSN ? 1 : 0;
  for (int i = 0; i < n_refs; ++i) {
    const ccpt_image& im = refs[i];
    const int code = shape_code(im.ny, im.nx);
    const size_t npx = (size_t)im.ny * im.nx, spec = spec_elems(code);
    const SizeTables& st = ctx->tables[table_key(code)];
    if ((size_t)i == ctx->refs.size()) ctx->refs.emplace_back();
    Ref& r = ctx->refs[i];
    if (r.n != code) {
      free_ref(r);
      r.n = code;
      if (!device_alloc(r.spec, spec * sizeof(float2)) || !device_alloc(r.img, npx * sizeof(float)) ||
          (fp64(ctx) && !device_alloc(r.spec64, spec * sizeof(double2))) ||
          (weight && !device_alloc(r.espec, spec * sizeof(float2))))
        return lost(CCPT_E_NOMEM, "reference spectra");
    }
    const int ny = code_ny(code), nx = code_nx(code), tr = code_trans(code);
    // the context's float copy is stored as given (pitch nx), a wide one read
    // transposed; CC-SN keeps F[E] too (held tall), the state of real-time
    // updates (B = -1/(E+eps) is not linear in E); the FP64 spectrum comes
    // from the reference's own values
    if (launch_ref_copy(im.data, im.dtype, im.pitch, im.ny, im.nx, r.img, s) ||
        launch_spectrum(ny, nx, r.img, CCPT_F32, im.nx, 0, tr, 1, weight, (float)ctx->o.eps, 1, T, r.spec,
                        st.tw, s) ||
        (weight && launch_spectrum(ny, nx, r.img, CCPT_F32, im.nx, 0, tr, 1, 0, 0.f, 0, T, r.espec, st.tw, s)) ||
        (fp64(ctx) && launch_spectrum64(im.nx, im.data, im.dtype, im.pitch, 0, 1, weight, ctx->o.eps, 1, T64,
                                        r.spec64, st.tw64, s)))
      return lost(CCPT_E_HIP, "reference spectrum launch failed");
  }
  HIP_CHECK(ctx, hipStreamSynchronize(s));
  return CCPT_OK;
}

int ccpt_track_batch(ccpt_ctx* ctx, const ccpt_roi* rois, int n, ccpt_result* out,
                     void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (n < 0 || (n > 0 && (!rois || !out))) return fail(ctx, CCPT_E_INVALID, "bad roi array");
  if (n == 0) return CCPT_OK;
  int rc = set_device(ctx);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  Plan plan;
  rc = plan_rois(ctx, rois, n, plan);
  if (rc) return rc;
  const std::vector<int>& sig = plan.sig;
  const int ngroups = (int)sig.size() / 2;
  // size groups on lanes: the most expensive first, each to the lane with the
  // least work so far (work = FFT flops and a term in the grid's size; FFT flops
  // alone spread 2048 ROIs of seven sizes worse, 483 us against 447); one lane
  // when profiling (stage timing follows one stream)
  const int want = ctx->lanes > 0 ? ctx->lanes : kMaxLanes;
  const int nl = (ctx->o.flags & CCPT_FLAG_PROFILE) ? 1 : std::max(1, std::min(ngroups, want));
  std::vector<int> lane_of(ngroups, 0);
  if (nl > 1) {
    std::vector<double> cost(ngroups), load(nl, 0.0);
    std::vector<int> order(ngroups);
    for (int gi = 0; gi < ngroups; ++gi) {
      const int nn = sig[2 * gi];
      const double ny = code_ny(nn), nx = code_nx(nn), h = nx / 2 + 1, m = ctx->M;
      cost[gi] = sig[2 * gi + 1] * (10.0 * ny * nx * std::log2(ny * nx) + 8.0 * m * ny * h + 4.0 * m * m * h);
      order[gi] = gi;
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
    for (int gi : order) {
      const int l = (int)(std::min_element(load.begin(), load.end()) - load.begin());
      lane_of[gi] = l;
      load[l] += cost[gi];
    }
  }
  // per-lane needs (one lane: per chunk slot, two slots when some group has
  // several chunks and two-stream chunks are on)
  std::vector<size_t> lws, lst, ows, ost;
  int nslots = 1;
  auto layout = [&](bool small) {
    lws.assign(nl, 0);
    lst.assign(nl, 0);
    nslots = 1;
    for (int gi = 0; gi < ngroups; ++gi) {
      const int nn = sig[2 * gi], cnt = sig[2 * gi + 1], l = lane_of[gi];
      const std::vector<Launch> ls = launches(ctx, nn, cnt, small, 0);
      const int chunk = largest(ls);
      lws[l] = std::max(lws[l], frame_ws_bytes(nn, ctx->o.precision) * (size_t)chunk + 256);
      lst[l] = std::max(lst[l], (size_t)chunk);
      if (nl == 1 && ls.size() > 1 && use_slots(ctx)) nslots = 2;
    }
    ows.assign(nl + 1, 0);
    ost.assign(nl + 1, 0);
    for (int l = 0; l < nl; ++l) {
      lws[l] = (lws[l] + 255) / 256 * 256;
      ows[l + 1] = ows[l] + lws[l] * nslots;
      ost[l + 1] = ost[l] + lst[l] * nslots;
    }
  };
  // a card with no room for the launches' workspace takes smaller ones
  layout(false);
  rc = ask_ws(ctx, ows[nl], s);
  const bool small = rc == CCPT_E_NOMEM;
  if (small) {
    layout(true);
    rc = ensure_ws(ctx, ows[nl]);
  }
  if (rc) return rc;
  rc = ensure_state(ctx, ost[nl], s);
  if (rc) return rc;
  rc = upload_desc(ctx, plan.desc, s);
  if (rc) return rc;

  std::vector<int> first(ngroups, 0);
  for (int gi = 1; gi < ngroups; ++gi) first[gi] = first[gi - 1] + sig[2 * gi - 1];
  std::vector<char> pairs(ngroups);
  for (int gi = 0; gi < ngroups; ++gi) pairs[gi] = pairs_ok(plan.desc, first[gi], sig[2 * gi + 1]);

  auto launch_all = [&]() -> int {
    // lanes 1.. start after everything already queued on the caller's stream
    if (nl > 1) {
      HIP_CHECK(ctx, hipEventRecord(ctx->fork_evt, s));
      for (int l = 1; l < nl; ++l) HIP_CHECK(ctx, hipStreamWaitEvent(ctx->lane_s[l - 1], ctx->fork_evt, 0));
    }
    int r2 = CCPT_OK;
    for (int l = 0; l < nl && r2 == CCPT_OK; ++l) {
      CallMem mem = ctx_mem(ctx);
      mem.ws = ctx->ws + ows[l];
      mem.slot_ws = lws[l];
      mem.st = ctx->st_buf + ost[l];
      mem.slot_st = lst[l];
      if (nl > 1) mem.slots = false;
      mem.small = small;
      hipStream_t ls = l ? ctx->lane_s[l - 1] : s;
      for (int gi = 0; gi < ngroups && r2 == CCPT_OK; ++gi) {
        if (lane_of[gi] != l) continue;
        const int nn = sig[2 * gi], cnt = sig[2 * gi + 1];
        r2 = run_group(ctx, mem, nn, ctx->d_desc, first[gi], cnt, out, ls, pairs[gi]);
      }
    }
    // every lane that was forked joins back, also after a failed launch
    for (int l = 1; l < nl; ++l) {
      if (hipEventRecord(ctx->lane_evt[l - 1], ctx->lane_s[l - 1]) != hipSuccess ||
          hipStreamWaitEvent(s, ctx->lane_evt[l - 1], 0) != hipSuccess) {
        (void)hipStreamSynchronize(ctx->lane_s[l - 1]);
        if (r2 == CCPT_OK) r2 = fail(ctx, CCPT_E_HIP, "joining lane %d failed", l);
      }
    }
    return r2;
  };

  const bool use_graph = (ctx->o.flags & CCPT_FLAG_GRAPH) && !(ctx->o.flags & CCPT_FLAG_PROFILE) &&
                         s != nullptr;
  if (!use_graph) return launch_all();
  GraphKey key{sig, pairs, small, out, s};
  auto it = ctx->graphs.find(key);
  if (it == ctx->graphs.end()) {
    hipGraph_t graph;
    HIP_CHECK(ctx, hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    int r2 = launch_all();
    hipError_t e = hipStreamEndCapture(s, &graph);
    if (r2) return r2;
    if (e != hipSuccess) return fail(ctx, CCPT_E_HIP, "capture: %s", hipGetErrorString(e));
    hipGraphExec_t exec;
    e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return fail(ctx, CCPT_E_HIP, "instantiate: %s", hipGetErrorString(e));
    it = ctx->graphs.emplace(key, exec).first;
  }
  HIP_CHECK(ctx, hipGraphLaunch(it->second, s));
  return CCPT_OK;
}

int ccpt_track_batch_static(ccpt_ctx* ctx, const ccpt_roi* rois, int n, ccpt_result* out,
                            void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (n < 0 || (n > 0 && (!rois || !out))) return fail(ctx, CCPT_E_INVALID, "bad roi array");
  if (n > CCPT_STATIC_MAX_ROIS)
    return fail(ctx, CCPT_E_INVALID, "%d rois exceed the static scratch's %d", n,
                CCPT_STATIC_MAX_ROIS);
  if (n == 0) return CCPT_OK;
  int rc = set_device(ctx);
  if (rc) return rc;
  char* base = (char*)scratch_ptr(ctx->device);
  if (!base) return fail(ctx, CCPT_E_HIP, "static scratch not set up on device %d", ctx->device);
  hipStream_t s = (hipStream_t)stream;
  Plan plan;
  rc = plan_rois(ctx, rois, n, plan);
  if (rc) return rc;
  // scratch layout: descriptors | frame states of one chunk | chunk workspace
  const size_t desc_bytes = ((size_t)n * sizeof(FrameDesc) + 255) / 256 * 256;
  constexpr size_t kStates = 4096;  // the most frames of a launch here (mem.slot_st limits it)
  const size_t st_bytes = (kStates * sizeof(FrameState) + 255) / 256 * 256;
  CallMem mem;
  mem.st = (FrameState*)(base + desc_bytes);
  mem.slot_st = kStates;
  mem.ws = base + desc_bytes + st_bytes;
  mem.chunk_bytes = kScratchBytes - desc_bytes - st_bytes;
  mem.slots = false;
  mem.mark = false;
  for (size_t gi = 0; gi < plan.sig.size(); gi += 2)
    if (frame_ws_bytes(plan.sig[gi], ctx->o.precision) > mem.chunk_bytes)
      return fail(ctx, CCPT_E_INVALID, "one %dx%d frame needs %zu bytes of workspace, more than "
                  "the static scratch holds", code_ny(plan.sig[gi]), code_nx(plan.sig[gi]),
                  frame_ws_bytes(plan.sig[gi], ctx->o.precision));
  FrameDesc* d_desc = (FrameDesc*)base;
  // from pageable memory: the host array is consumed before the call returns
  HIP_CHECK(ctx, hipMemcpyAsync(d_desc, plan.desc.data(), (size_t)n * sizeof(FrameDesc),
                                hipMemcpyHostToDevice, s));
  // whatever an earlier call left in the states: back to the initial state
  if (launch_init_state(mem.st, (int)kStates, s))
    return fail(ctx, CCPT_E_HIP, "state initialisation launch failed");
  int first = 0;
  for (size_t gi = 0; gi < plan.sig.size(); gi += 2) {
    const int nn = plan.sig[gi], cnt = plan.sig[gi + 1];
    rc = run_group(ctx, mem, nn, d_desc, first, cnt, out, s, pairs_ok(plan.desc, first, cnt));
    if (rc) return rc;
    first += cnt;
  }
  return CCPT_OK;
}

int ccpt_track_grad(ccpt_ctx* ctx, const ccpt_roi* rois, int n, const ccpt_result* fwd,
                    const double* g_d, const double* g_peak, float* g_frames, float* g_ref,
                    void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (n < 0 || (n > 0 && (!rois || !fwd || !g_d)))
    return fail(ctx, CCPT_E_INVALID, "bad gradient arguments");
  if (!g_frames && !g_ref) return CCPT_OK;
  int rc = set_device(ctx);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (n == 0) {
    // no rois: every reference gradient is an empty sum
    size_t total = 0;
    for (const Ref& r : ctx->refs) total += (size_t)code_ny(r.n) * code_nx(r.n);
    if (g_ref && total && launch_zero(g_ref, total * sizeof(float), s))
      return fail(ctx, CCPT_E_HIP, "zero launch failed");
    return CCPT_OK;
  }
  for (int i = 0; i < n; ++i) {
    rc = require_square(ctx, rois[i].ny, rois[i].nx, "ccpt_track_grad");
    if (rc) return rc;
  }
  Plan plan;
  rc = plan_rois(ctx, rois, n, plan, true);
  if (rc) return rc;
  const int nrefs = (int)ctx->refs.size();
  // packed offsets of the frame gradients (roi order) and of the reference gradients
  std::vector<long> goff(n);
  long acc_el = 0;
  for (int i = 0; i < n; ++i) {
    goff[i] = acc_el;
    acc_el += (long)rois[i].ny * rois[i].nx;
  }
  std::vector<long> roff(nrefs), aoff(nrefs);
  long ro = 0, ao = 0;
  for (int r = 0; r < nrefs; ++r) {
    const int nn = ctx->refs[r].n;
    roff[r] = ro;
    ro += (long)nn * nn;
    aoff[r] = ao;
    ao += (long)spec_elems(nn);
  }
  // Workspace: QB of a chunk's frames, and T, F[A], QA and an image of those that
  // the passes take: all, or where frames fit LDS at most a short last round (so
  // that 1024 frames of 128 x 128 are one launch; in launches of 795 and 229, with
  // room for the passes of all, the adjoint took 165 us instead of 136).
  const size_t budget = (size_t)256 << 20;
  auto in_lds = [](int nn) { return lds_frames(nn, nn, kLdsRound) > 0; };
  auto qb_bytes = [](int nn) { return spec_elems(nn) * sizeof(float2); };
  auto pass_bytes = [](int nn) { return 3 * spec_elems(nn) * sizeof(float2) + (size_t)nn * nn * 4; };
  auto chunk_of = [&](int nn, int cnt) {
    const size_t fit = in_lds(nn) ? (budget - pass_bytes(nn) * (kGradMinFrames - 1)) / qb_bytes(nn)
                                  : budget / (qb_bytes(nn) + pass_bytes(nn));
    return std::max(1, (int)std::min<size_t>({(size_t)cnt, fit, (size_t)65535}));  // (a grid's y)
  };
  auto pass_frames = [&](int nn, int chunk) { return in_lds(nn) ? std::min(chunk, kGradMinFrames - 1) : chunk; };
  size_t ws_need = 0, img_need = 0;
  for (size_t gi = 0; gi < plan.sig.size(); gi += 2) {
    const int nn = plan.sig[gi], chunk = chunk_of(nn, plan.sig[gi + 1]);
    ws_need = std::max(ws_need, qb_bytes(nn) * chunk + pass_bytes(nn) * pass_frames(nn, chunk) + 256);
  }
  for (int r = 0; r < nrefs; ++r)
    img_need = std::max(img_need, pass_bytes(ctx->refs[r].n) + 256);
  rc = ensure_ws(ctx, std::max(ws_need, img_need));
  if (rc) return rc;
  // frames of each chunk by reference, in runs (the sums of the reference gradients)
  struct ChunkSums {
    int order, run, nruns, head, nheads;
  };
  std::vector<int> order;
  std::vector<int2> runs;
  std::vector<int4> heads;
  std::vector<ChunkSums> sums;
  if (g_ref) {
    int first = 0;
    for (size_t gi = 0; gi < plan.sig.size(); gi += 2) {
      const int nn = plan.sig[gi], cnt = plan.sig[gi + 1];
      const int chunk = chunk_of(nn, cnt);
      for (int c0 = 0; c0 < cnt; c0 += chunk) {
        const int count = std::min(chunk, cnt - c0);
        const FrameDesc* d = plan.desc.data() + first + c0;
        ChunkSums cs{(int)order.size(), (int)runs.size(), 0, (int)heads.size(), 0};
        for (int i = 0; i < count; ++i) order.push_back(i);
        int* o = order.data() + cs.order;
        std::stable_sort(o, o + count, [&](int x, int y) { return d[x].ref_id < d[y].ref_id; });
        for (int i = 0; i < count;) {
          const int ref = d[o[i]].ref_id, run0 = (int)runs.size() - cs.run;
          int e = i;
          while (e < count && d[o[e]].ref_id == ref) ++e;
          for (; i < e; i += kSumRun) runs.push_back(int2{i, std::min(kSumRun, e - i)});
          i = e;
          heads.push_back(int4{ref, run0, (int)runs.size() - cs.run - run0, 0});
        }
        cs.nruns = (int)runs.size() - cs.run;
        cs.nheads = (int)heads.size() - cs.head;
        sums.push_back(cs);
      }
      first += cnt;
    }
  }
  // the small tables, in order of alignment
  const size_t o_runs = heads.size() * sizeof(int4), o_goff = o_runs + runs.size() * sizeof(int2);
  const size_t o_acc = o_goff + (size_t)n * sizeof(long), o_order = o_acc + (size_t)nrefs * sizeof(void*);
  const size_t small_bytes = o_order + order.size() * sizeof(int);
  rc = ensure_buf(ctx, ctx->gsmall, ctx->gsmall_cap, small_bytes);
  if (rc) return rc;
  if (g_ref) {
    rc = ensure_buf(ctx, ctx->acc_buf, ctx->acc_cap, (size_t)ao * sizeof(float2));
    if (rc) return rc;
  }
  rc = upload_desc(ctx, plan.desc, s);
  if (rc) return rc;
  // small table upload through pinned staging
  HIP_CHECK(ctx, hipEventSynchronize(ctx->small_evt));
  if (small_bytes > ctx->h_small_cap) {
    if (ctx->h_small) (void)hipHostFree(ctx->h_small);
    ctx->h_small = nullptr;
    ctx->h_small_cap = 0;
    if (!pinned_alloc(ctx->h_small, small_bytes))
      return fail(ctx, CCPT_E_NOMEM, "pinned staging");
    ctx->h_small_cap = small_bytes;
  }
  if (g_ref) {
    memcpy(ctx->h_small, heads.data(), heads.size() * sizeof(int4));
    memcpy(ctx->h_small + o_runs, runs.data(), runs.size() * sizeof(int2));
    memcpy(ctx->h_small + o_order, order.data(), order.size() * sizeof(int));
  }
  memcpy(ctx->h_small + o_goff, goff.data(), (size_t)n * sizeof(long));
  float2** accp = (float2**)(ctx->h_small + o_acc);
  for (int r = 0; r < nrefs; ++r)
    accp[r] = g_ref ? (float2*)ctx->acc_buf + aoff[r] : nullptr;
  HIP_CHECK(ctx, hipMemcpyAsync(ctx->gsmall, ctx->h_small, small_bytes, hipMemcpyHostToDevice, s));
  HIP_CHECK(ctx, hipEventRecord(ctx->small_evt, s));
  const char* small = (const char*)ctx->gsmall;
  const long* d_goff = (const long*)(small + o_goff);
  float2* const* d_acc = (float2* const*)(small + o_acc);
  if (g_ref && launch_zero(ctx->acc_buf, (size_t)ao * sizeof(float2), s))
    return fail(ctx, CCPT_E_HIP, "zero launch failed");

  const Marker mark = marker_of(ctx, s);
  const int mode = ctx->o.mode;
  const float eps = (float)ctx->o.eps;
  int first = 0, chunk_no = 0;
  mark(CCPT_STAGE_GRAD, 1);
  for (size_t gi = 0; gi < plan.sig.size(); gi += 2) {
    const int nn = plan.sig[gi], cnt = plan.sig[gi + 1];
    const int chunk = chunk_of(nn, cnt);
    const float2* tw = ctx->tables[nn].tw;
    const size_t spec = spec_elems(nn);
    for (int c0 = 0; c0 < cnt; c0 += chunk) {
      const int count = std::min(chunk, cnt - c0);
      const size_t pf = pass_frames(nn, chunk);
      float2* QB = (float2*)ctx->ws;
      float2* T = QB + spec * chunk;
      float2* FA = T + spec * pf;
      float2* QA = FA + spec * pf;
      float* img = (float*)(QA + spec * pf);
      const int f0 = first + c0;
      GradParams g{ctx->d_desc, f0, count, fwd, g_d, g_peak, g_ref ? QB : nullptr, d_goff, g_frames, mode, eps, tw};
      // frames that fit LDS in one kernel, the others in passes
      const int nl = lds_frames(nn, nn, count, kGradMinFrames);
      g.count = nl;
      if (nl > 0 && launch_grad_lds(nn, g, s)) return fail(ctx, CCPT_E_HIP, "gradient launch failed");
      if (nl < count) {
        g.first = f0 + nl;
        g.count = count - nl;
        if (g_ref) g.QB = QB + spec * nl;
        if ((g_ref && launch_frame_spectra(nn, ctx->d_desc, g.first, g.count, mode, eps, T, FA, tw, s)) ||
            launch_grad_psi(nn, g, FA, QA, s))
          return fail(ctx, CCPT_E_HIP, "gradient launch failed");
        if (g_frames && (launch_inverse(nn, QA, g.count, 2.0f, T, img, tw, s) ||
                         launch_grad_frames(nn, ctx->d_desc, g.first, g.count, img, d_goff, g_frames, mode,
                                            eps, s)))
          return fail(ctx, CCPT_E_HIP, "frame gradient launch failed");
      }
      if (g_ref) {
        const ChunkSums& cs = sums[chunk_no++];
        const RefSums t{(const int*)(small + o_order) + cs.order, (const int2*)(small + o_runs) + cs.run,
                        (const int4*)small + cs.head, cs.nruns, cs.nheads};
        if (launch_ref_accum(nn, QB, t, d_acc, s))
          return fail(ctx, CCPT_E_HIP, "reference gradient launch failed");
      }
    }
    first += cnt;
  }
  if (g_ref) {
    for (int r = 0; r < nrefs; ++r) {
      const int nn = ctx->refs[r].n;
      float2* T = (float2*)ctx->ws;
      float* img = (float*)(T + spec_elems(nn));
      if (launch_inverse(nn, (float2*)ctx->acc_buf + aoff[r], 1, 2.0f, T, img, ctx->tables[nn].tw,
                         s) ||
          launch_grad_ref_chain(img, ctx->refs[r].img, nn * nn, mode, eps, g_ref + roff[r], s))
        return fail(ctx, CCPT_E_HIP, "reference gradient launch failed");
    }
  }
  mark(CCPT_STAGE_GRAD, 0);
  return CCPT_OK;
}

int ccpt_fisher(ccpt_ctx* ctx, const ccpt_image* mu, double* fisher, void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (!mu || !fisher) return fail(ctx, CCPT_E_INVALID, "null argument");
  int rc = check_image(ctx, mu->data, mu->ny, mu->nx, mu->pitch, mu->dtype, "mean image", 0);
  if (!rc) rc = require_square(ctx, mu->ny, mu->nx, "ccpt_fisher");
  if (rc) return rc;
  rc = set_device(ctx);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  const int n = mu->nx;
  HIP_CHECK(ctx, hipStreamSynchronize(s));
  {
    std::vector<char> raw(((size_t)(mu->ny - 1) * mu->pitch + mu->nx) * dtype_bytes(mu->dtype));
    HIP_CHECK(ctx, hipMemcpy(raw.data(), mu->data, raw.size(), hipMemcpyDeviceToHost));
    for (int y = 0; y < n; ++y)
      for (int x = 0; x < n; ++x) {
        const double v = pixel(raw.data(), mu->dtype, (size_t)y * mu->pitch + x);
        if (!(v > 0.0) || !std::isfinite(v))
          return fail(ctx, CCPT_E_INVALID, "mean image must be > 0 and finite (%d, %d)", y, x);
      }
  }
  rc = ensure_tables(ctx, n);
  if (rc) return rc;
  const size_t spec = spec_elems(n);
  const int nblocks = 64;
  const size_t bytes = 4 * spec * sizeof(float2) + 2 * (size_t)n * n * sizeof(float) +
                       (size_t)nblocks * 3 * sizeof(double) + 256;
  char* tmp = nullptr;
  HIP_CHECK(ctx, hipMalloc(&tmp, bytes));
  float2* F = (float2*)tmp;
  float2* Dy = F + spec;
  float2* Dx = Dy + spec;
  float2* T = Dx + spec;
  float* iy = (float*)(T + spec);
  float* ix = iy + (size_t)n * n;
  double* part = (double*)(((uintptr_t)(ix + (size_t)n * n) + 15) & ~(uintptr_t)15);
  const float2* tw = ctx->tables[n].tw;
  int bad = launch_spectrum(n, n, mu->data, mu->dtype, mu->pitch, 0, 0, 1, 0, 0.f, 0, T, F, tw,
                            s) ||
            launch_fisher_deriv(n, F, Dy, Dx, s) || launch_inverse(n, Dy, 1, 2.0f, T, iy, tw, s) ||
            launch_inverse(n, Dx, 1, 2.0f, T, ix, tw, s) ||
            launch_fisher_reduce(iy, ix, mu->data, mu->dtype, mu->pitch, n, part, nblocks, fisher, s);
  hipError_t e = hipStreamSynchronize(s);
  (void)hipFree(tmp);
  if (bad) return fail(ctx, CCPT_E_HIP, "fisher launch failed");
  if (e != hipSuccess) return fail(ctx, CCPT_E_HIP, "fisher: %s", hipGetErrorString(e));
  return CCPT_OK;
}

int ccpt_mean_aligned(ccpt_ctx* ctx, const ccpt_roi* rois, int n, const ccpt_result* fwd,
                      float* out, void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (n < 1 || !rois || !fwd || !out) return fail(ctx, CCPT_E_INVALID, "bad arguments");
  int rc = set_device(ctx);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  const int N = rois[0].nx;
  std::vector<FrameDesc> desc(n);
  for (int i = 0; i < n; ++i) {
    const ccpt_roi& r = rois[i];
    rc = check_image(ctx, r.data, r.ny, r.nx, r.pitch, r.dtype, "roi", i);
    if (!rc) rc = require_square(ctx, r.ny, r.nx, "ccpt_mean_aligned");
    if (rc) return rc;
    if (r.nx != N) return fail(ctx, CCPT_E_INVALID, "roi %d: size %d differs from %d", i, r.nx, N);
    desc[i] = FrameDesc{r.data, nullptr, r.pitch, r.dtype, i, 0};
  }
  rc = ensure_tables(ctx, N);
  if (rc) return rc;
  const size_t spec = spec_elems(N);
  const size_t per_frame = 2 * spec * sizeof(float2);  // T and the frame's spectrum
  const int chunk = std::max(1, std::min<int>(n, (int)(((size_t)256 << 20) / per_frame)));
  const size_t head = spec * sizeof(float2) + 256;  // accumulator, counter
  rc = ensure_ws(ctx, head + per_frame * chunk);
  if (rc) return rc;
  rc = upload_desc(ctx, desc, s);
  if (rc) return rc;
  float2* acc = (float2*)ctx->ws;
  unsigned* cnt = (unsigned*)(acc + spec);
  float2* T = (float2*)((char*)ctx->ws + head);
  float2* F = T + spec * chunk;
  const float2* tw = ctx->tables[N].tw;
  if (launch_zero(acc, head, s)) return fail(ctx, CCPT_E_HIP, "zero launch failed");
  for (int c0 = 0; c0 < n; c0 += chunk) {
    const int count = std::min(chunk, n - c0);
    // frames that fit LDS in one kernel, the others in passes
    const int nl = lds_frames(N, N, count), rest = count - nl;
    float2* Fr = F + spec * nl;
    if ((nl > 0 && launch_align_lds(N, ctx->d_desc, c0, nl, fwd, tw, F, cnt, s)) ||
        (rest > 0 &&
         (launch_frame_spectra(N, ctx->d_desc, c0 + nl, rest, CCPT_MODE_CCU, 0.f, T, Fr, tw, s) ||
          launch_align(N, ctx->d_desc, c0 + nl, rest, fwd, Fr, cnt, s))) ||
        launch_sum_spectra(N, count, F, acc, s))
      return fail(ctx, CCPT_E_HIP, "alignment launch failed");
  }
  // the row pass of the inverse returns half the unnormalised transform
  if (launch_inverse(N, acc, 1, 2.0f / ((float)N * (float)N), T, out, tw, s) ||
      launch_scale_by_count(out, N * N, 1.0f, cnt, s))
    return fail(ctx, CCPT_E_HIP, "inverse launch failed");
  return CCPT_OK;
}

int ccpt_track_update(ccpt_ctx* ctx, const ccpt_roi* roi, double a0, ccpt_result* out,
                      void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (!roi || !out || !(a0 >= 0.0 && a0 <= 1.0))
    return fail(ctx, CCPT_E_INVALID, "bad arguments");
  if (fp64(ctx)) return fail(ctx, CCPT_E_UNSUPPORTED, "real-time updates need FP32 or BF16X2 precision");
  int rc = ccpt_track_batch(ctx, roi, 1, out, stream);  // validates roi and reference id
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  Ref& R = ctx->refs[roi->ref_id];
  const int code = R.n;
  const int ny = code_ny(code), nx = code_nx(code), tr = code_trans(code);
  const size_t spec = spec_elems(code);
  // (the context's copy of a rectangle's E is read by nothing: the adjoint
  // takes square frames only)
  rc = ensure_buf(ctx, ctx->rt_buf, ctx->rt_cap, spec * sizeof(float2));
  if (rc) return rc;
  const bool sn = ctx->o.mode == CCPT_MODE_CCSN;
  // (track_batch left the frame's descriptor at index 0)
  const RtUpdate u{ctx->d_desc, out, (float2*)ctx->rt_buf, R.spec, sn ? R.espec : nullptr,
                   is_rect(code) ? nullptr : R.img, (float)a0, (float)(1.0 - a0), (float)ctx->o.eps,
                   ctx->tables[table_key(code)].tw};
  if (launch_rt_update(ny, nx, tr, u, s)) return fail(ctx, CCPT_E_HIP, "reference update launch failed");
  return CCPT_OK;
}

int ccpt_drift_filter(const double* r, int n, double a0, double rate_limit, double* state,
                      double* out) {
  if (n < 0 || (n > 0 && (!r || !out)) || !state || !(a0 >= 0.0 && a0 <= 1.0) ||
      !(rate_limit >= 0.0) || !(state[2] >= 0.0))
    return CCPT_E_INVALID;
  const double b1 = 1.0 - a0;
  double Ry = state[0], Rx = state[1];
  bool first = state[2] == 0.0;
  for (int i = 0; i < n; ++i) {
    const double ry = r[2 * i], rx = r[2 * i + 1];
    if (first) {  // Eq. 10 with R_{-1} = 0: R_0 = a0 r_0, never rate-limited
      Ry = a0 * ry;
      Rx = a0 * rx;
      first = false;
    } else if (rate_limit > 0.0) {  // Eq. 11-12
      double dy = a0 * ry + (b1 - 1.0) * Ry, dx = a0 * rx + (b1 - 1.0) * Rx;
      const double L = std::hypot(dy, dx);
      if (L > rate_limit) {
        dy *= rate_limit / L;
        dx *= rate_limit / L;
      }
      Ry += dy;
      Rx += dx;
    } else {  // Eq. 10
      Ry = a0 * ry + b1 * Ry;
      Rx = a0 * rx + b1 * Rx;
    }
    out[2 * i] = ry - Ry;
    out[2 * i + 1] = rx - Rx;
  }
  state[0] = Ry;
  state[1] = Rx;
  state[2] += (double)n;
  return CCPT_OK;
}

int ccpt_stage_times(ccpt_ctx* ctx, double* ms, int* launches, int n_stages, int reset) {
  if (!ctx || n_stages < 0 || (n_stages > 0 && (!ms || !launches))) return CCPT_E_INVALID;
  for (int i = 0; i < n_stages; ++i) {
    ms[i] = 0.0;
    launches[i] = 0;
  }
  for (auto& sp : ctx->spans) {
    HIP_CHECK(ctx, hipEventSynchronize(sp.b));
    float t = 0.f;
    HIP_CHECK(ctx, hipEventElapsedTime(&t, sp.a, sp.b));
    if (sp.stage >= 0 && sp.stage < n_stages) {
      ms[sp.stage] += t;
      launches[sp.stage] += 1;
    }
  }
  if (reset) {
    for (auto& sp : ctx->spans) {
      ctx->ev_pool.push_back(sp.a);
      ctx->ev_pool.push_back(sp.b);
    }
    ctx->spans.clear();
  }
  return CCPT_OK;
}

// Event-timed average of `reps` calls of ccpt_track_batch (one untimed call
// first: allocations and graph captures); a negative value if a call failed.
static float time_batch(ccpt_ctx* ctx, const ccpt_roi* rois, int n, ccpt_result* out,
                        void* stream, hipEvent_t e0, hipEvent_t e1, int reps) {
  hipStream_t s = (hipStream_t)stream;
  if (ccpt_track_batch(ctx, rois, n, out, stream) != CCPT_OK) return -1.f;
  if (hipEventRecord(e0, s) != hipSuccess) return -1.f;
  for (int r = 0; r < reps; ++r)
    if (ccpt_track_batch(ctx, rois, n, out, stream) != CCPT_OK) return -1.f;
  float ms = 0.f;
  if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
      hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
    return -1.f;
  return ms / reps;
}

// Coordinate search over the launch plan of one shape code: chunk sizes, then
// the block plans that apply to the shape (the threshold of the split window
// expansion; for 256x256 the one-kernel correlation's), then chunk sizes again if
// a block plan changed; every candidate timed on the whole call.
static void tune_shape(ccpt_ctx* ctx, int code, int count, const ccpt_roi* rois, int n,
                       ccpt_result* out, void* stream, hipEvent_t e0, hipEvent_t e1,
                       float& best_ms) {
  Schedule& sc = ctx->sched[code];
  auto trial = [&](Schedule cand) {
    const Schedule keep = sc;
    sc = cand;
    drop_graphs(ctx);
    const float ms = time_batch(ctx, rois, n, out, stream, e0, e1, 3);
    if (ms >= 0.f && ms < best_ms) {
      best_ms = ms;
      return true;
    }
    sc = keep;
    return false;
  };
  const int cands[] = {16, 32, 64, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048, 4096};
  auto sweep_chunks = [&]() {
    for (int c : cands) {
      if (c > count && c != cands[0]) break;
      if (frame_ws_bytes(code, ctx->o.precision) * (size_t)std::min(c, count) > ((size_t)8 << 30))
        break;
      Schedule cand = sc;
      cand.chunk = c;
      (void)trial(cand);
    }
  };
  sweep_chunks();
  bool changed = false;
  for (int sb : {0, kSplitBlocks, 512}) {
    Schedule cand = sc;
    cand.split_blocks = sb;
    changed |= trial(cand);
  }
  if (code_ny(code) == 256 && code_nx(code) == 256 && !fp64(ctx))
    for (int fm : {1, kFusedMinFrames, 1 << 30}) {
      Schedule cand = sc;
      cand.fused_min = fm;
      changed |= trial(cand);
    }
  if (changed) sweep_chunks();
}

int ccpt_autotune(ccpt_ctx* ctx, int n, int batch, void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (batch < 1 || !supported_size(n)) return fail(ctx, CCPT_E_INVALID, "bad tuning shape");
  int rid = -1;
  for (int r = 0; r < (int)ctx->refs.size(); ++r)
    if (ctx->refs[r].n == n) {
      rid = r;
      break;
    }
  if (rid < 0) return fail(ctx, CCPT_E_NOREF, "no reference of size %d to tune with", n);
  int rc = set_device(ctx);
  if (rc) return rc;
  // every tuning frame is the reference image itself (timing does not depend on content)
  std::vector<ccpt_roi> rois(batch);
  for (auto& r : rois) r = ccpt_roi{ctx->refs[rid].img, n, n, n, CCPT_F32, rid};
  ccpt_result* out = nullptr;
  HIP_CHECK(ctx, hipMalloc(&out, (size_t)batch * sizeof(ccpt_result)));
  hipEvent_t e0, e1;
  HIP_CHECK(ctx, hipEventCreate(&e0));
  HIP_CHECK(ctx, hipEventCreate(&e1));
  const int saved_flags = ctx->o.flags;
  ctx->o.flags = 0;  // no graphs or profiling while tuning
  ctx->sched[n] = Schedule{};
  // the default launches first: no chunk stands for them (they may be one launch
  // where every chunk makes two), and a candidate has to beat them
  drop_graphs(ctx);
  float best = time_batch(ctx, rois.data(), batch, out, stream, e0, e1, 3);
  if (best < 0.f) best = 1e30f;
  tune_shape(ctx, n, batch, rois.data(), batch, out, stream, e0, e1, best);
  ctx->o.flags = saved_flags;
  drop_graphs(ctx);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipFree(out);
  ctx->last_desc.clear();
  return CCPT_OK;
}

int ccpt_autotune_batch(ccpt_ctx* ctx, const ccpt_roi* rois, int n, void* stream) {
  if (!ctx) return CCPT_E_INVALID;
  if (n < 1 || !rois) return fail(ctx, CCPT_E_INVALID, "bad roi array");
  int rc = set_device(ctx);
  if (rc) return rc;
  Plan plan;
  rc = plan_rois(ctx, rois, n, plan);  // validates every roi
  if (rc) return rc;
  ccpt_result* out = nullptr;
  HIP_CHECK(ctx, hipMalloc(&out, (size_t)n * sizeof(ccpt_result)));
  hipEvent_t e0, e1;
  HIP_CHECK(ctx, hipEventCreate(&e0));
  HIP_CHECK(ctx, hipEventCreate(&e1));
  const int saved_flags = ctx->o.flags;
  ctx->o.flags = 0;  // no graphs or profiling while tuning
  const int ngroups = (int)plan.sig.size() / 2;
  auto tune_lanes = [&](float& best) {
    int best_l = ctx->lanes;
    for (int l = 1; l <= std::min(ngroups, kMaxLanes); ++l) {
      ctx->lanes = l;
      drop_graphs(ctx);
      const float ms = time_batch(ctx, rois, n, out, stream, e0, e1, 3);
      if (ms >= 0.f && ms < best) {
        best = ms;
        best_l = l;
      }
    }
    ctx->lanes = best_l;
  };
  float best = 1e30f;
  for (int gi = 0; gi < ngroups; ++gi) ctx->sched[plan.sig[2 * gi]] = Schedule{};
  ctx->lanes = 0;
  tune_lanes(best);
  // the shapes in the call's order (largest frames first), each plan timed on
  // the whole call with the others' plans fixed
  for (int gi = 0; gi < ngroups; ++gi)
    tune_shape(ctx, plan.sig[2 * gi], plan.sig[2 * gi + 1], rois, n, out, stream, e0, e1, best);
  tune_lanes(best);
  ctx->o.flags = saved_flags;
  drop_graphs(ctx);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipFree(out);
  ctx->last_desc.clear();
  return CCPT_OK;
}

int ccpt_schedule(ccpt_ctx* ctx, int n, int* chunk, int set) {
  if (!ctx || !chunk) return CCPT_E_INVALID;
  if (!supported_size(n)) return fail(ctx, CCPT_E_UNSUPPORTED, "size %d", n);
  if (set) {
    if (*chunk < 0 || *chunk > (1 << 20)) return fail(ctx, CCPT_E_INVALID, "chunk %d", *chunk);
    ctx->sched[n].chunk = *chunk;
    drop_graphs(ctx);
  } else {
    *chunk = chunk_for(ctx, n);
  }
  return CCPT_OK;
}

int ccpt_get_plan(ccpt_ctx* ctx, int ny, int nx, ccpt_plan* p) {
  if (!ctx || !p) return CCPT_E_INVALID;
  const int code = shape_code(ny, nx);
  if (!code) return fail(ctx, CCPT_E_UNSUPPORTED, "shape %dx%d", ny, nx);
  p->chunk = chunk_for(ctx, code);
  p->split_blocks = split_blocks_for(ctx, code);
  p->fused_min = fused_min_for(ctx, code);
  return CCPT_OK;
}

int ccpt_set_plan(ccpt_ctx* ctx, int ny, int nx, const ccpt_plan* p) {
  if (!ctx || !p) return CCPT_E_INVALID;
  const int code = shape_code(ny, nx);
  if (!code) return fail(ctx, CCPT_E_UNSUPPORTED, "shape %dx%d", ny, nx);
  if (p->chunk < 0 || p->chunk > (1 << 20) || p->split_blocks < -1 || p->split_blocks > 512 ||
      p->fused_min < -1)
    return fail(ctx, CCPT_E_INVALID, "plan {%d, %d, %d}", p->chunk, p->split_blocks, p->fused_min);
  Schedule& sc = ctx->sched[code];
  sc.chunk = p->chunk;
  sc.split_blocks = p->split_blocks;
  sc.fused_min = p->fused_min;
  drop_graphs(ctx);
  return CCPT_OK;
}

int ccpt_lanes(ccpt_ctx* ctx, int* lanes, int set) {
  if (!ctx || !lanes) return CCPT_E_INVALID;
  if (set) {
    if (*lanes < 0 || *lanes > kMaxLanes) return fail(ctx, CCPT_E_INVALID, "lanes %d", *lanes);
    ctx->lanes = *lanes;
    drop_graphs(ctx);
  } else {
    *lanes = ctx->lanes > 0 ? ctx->lanes : kMaxLanes;
  }
  return CCPT_OK;
}

}  // extern "C"
