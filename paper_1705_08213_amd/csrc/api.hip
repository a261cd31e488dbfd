// api.hip -- the C ABI declared in include/ccc.h: argument validation, the
// per-device workspace, and dispatch to the kernels.
//
// Validation is pure host logic and runs before any HIP call, so every error
// path returns with nothing enqueued and outputs untouched.
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <stdlib.h>

#include <algorithm>
#include <atomic>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "../../include/ccc.h"
#include "kernels.h"
#include "many.h"

namespace {

constexpr int64_t kInt32Max = 2147483647;
// Largest row stride: the kernels address a 16-row block of the input with
// 32-bit byte offsets (15 ld + 64 < 2^32).
constexpr int64_t kMaxLd = int64_t(1) << 28;
// Largest row count whose complete-data Gram matrix (4 B per entry) the
// 3-way MFMA path keeps in the workspace (4 GiB); beyond it every unit takes
// the general path.
constexpr int64_t kGramMaxRows = 32768;

// Most operands (operands.hip) that the library holds on a device, over all
// its workspaces and batches; $CCC_OPERAND_LIMIT (bytes) overrides it.  They
// also never take more than half of the memory that is free.  Where they find
// no room the fp4 kernels read the packed rows.  That takes large calls up to
// 1.4 times as long (few rows of long fields, whose operands are small, up to
// eight times), but a wait for the device and other streams' buffers given
// back and allocated again would cost every call of a card that is nearly full
// milliseconds, and hold up everyone else's.  The check is one query of the
// free memory (5 us), made only when a buffer has to grow.
constexpr int64_t kOperandLimit = int64_t(16) << 30;

// Workspaces: one buffer per (device, stream) for eager calls, so that calls
// on different streams never share scratch, and one per (device, stream,
// capture) for captured calls: a graph may be replayed on any stream, beside
// other graphs captured on the same one and beside eager calls there, so it
// shares its scratch with neither.  A call holds g_mu while it enqueues its
// kernels, so that calls of several threads on one stream do not interleave.
// A graph holds the address of its buffers: they stay until the graph and its
// executables are destroyed, which a user object of the graph tells (`gone`).
// What such an executable last launched may still run, so the buffers are
// freed behind a wait, by a later eager call that finds more than kMaxGone of
// them, or more than kMaxGoneBytes, or runs out of memory.
struct Workspace {
  int dev = 0;
  hipStream_t stream = nullptr;
  size_t thread = 0;  // of hipStreamPerThread, which names a stream per thread
  unsigned long long capture = 0;  // id of the capture it belongs to, 0: eager calls
  std::shared_ptr<std::atomic<bool>> gone;  // of a capture: its graph is no more
  void* ptr = nullptr;  // what every call needs: flag, counts, Gram matrix
  size_t bytes = 0;
  void* ops = nullptr;  // operands and split tiles' sums, if they have room
  size_t ops_bytes = 0;
  uint64_t last_use = 0;
};
constexpr size_t kMaxGone = 8, kMaxGoneBytes = size_t(1) << 30;
// Workspaces of eager calls per device.  A framework's stream pool has 32
// streams; one past the bound waits for the device and gives back the half that
// was used longest ago, so that a program which makes streams without end waits
// once in 64 of them.
constexpr size_t kMaxWorkspaces = 128;

std::mutex g_mu;
std::vector<Workspace> g_ws;
std::vector<Workspace> g_retired;  // outgrown by a capture that may hold their address
std::map<int, int64_t> g_batch_operands;  // held by ccc_2way_many's batches, by device
uint64_t g_clock = 0;

// Identity of a call in the complete-data flag (Pair2Args::flag).
std::atomic<unsigned long long> g_call{1};

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int resolve_opts(const ccc_opts* opts, ccc_opts* out) {
  *out = ccc_default_opts();
  if (!opts) return CCC_OK;
  if (opts->path < CCC_PATH_AUTO || opts->path > CCC_PATH_MFMA) return CCC_ERR_ARG;
  if (!isfinite(opts->gamma)) return CCC_ERR_ARG;
  if (opts->flags & ~(unsigned)(CCC_ACCUMULATE | CCC_FINALIZE)) return CCC_ERR_ARG;
  if (opts->operands != CCC_OPERANDS_AUTO && opts->operands != CCC_OPERANDS_FP4 &&
      opts->operands != CCC_OPERANDS_INT8)
    return CCC_ERR_ARG;
  if (opts->path == CCC_PATH_POPCOUNT && opts->operands != CCC_OPERANDS_AUTO) return CCC_ERR_ARG;
  *out = *opts;
  return CCC_OK;
}

// fp4 operands for an MFMA call whose largest per-call field count is n_f
// (1), int8 (0), or CCC_ERR_RANGE when fp4 is forced beyond its exact range.
int use_fp4(const ccc_opts& o, int64_t n_f) {
  if (o.operands == CCC_OPERANDS_INT8) return 0;
  if (o.operands == CCC_OPERANDS_FP4) return n_f <= ccc::kF4MaxFields ? 1 : CCC_ERR_RANGE;
  return n_f <= ccc::kF4MaxFields ? 1 : 0;
}

// Table entries are at most 4 n_f (2-way) or 8 n_f (3-way): `mult` = 4 or 8.
// Compared by division first, so that no product of a huge n_f overflows.
bool fields_in_range(int64_t n_f, int64_t mult) { return n_f <= kInt32Max / mult; }

size_t round256(size_t bytes) { return (bytes + 255) / 256 * 256; }

int check_input(const uint8_t* v, int64_t n, int64_t n_f, int64_t ld) {
  if (n < 0 || n_f < 0 || ld < 0) return CCC_ERR_ARG;
  if (n > kInt32Max) return CCC_ERR_ARG;
  if (ld % 16 != 0) return CCC_ERR_ALIGN;
  if (ld > kMaxLd) return CCC_ERR_RANGE;
  if (n_f / 4 >= ld + (n_f % 4 == 0)) return CCC_ERR_ARG;  // ld < ceil(n_f/4), overflow-free
  if (n > 0 && !v) return CCC_ERR_ARG;
  if (v && !aligned16(v)) return CCC_ERR_ALIGN;
  return CCC_OK;
}

}  // namespace

namespace ccc {

int64_t operand_limit() {
  const char* env = getenv("CCC_OPERAND_LIMIT");
  return env && *env ? atoll(env) : kOperandLimit;
}

namespace {

// Id of the capture that `stream` is part of (its forks have the same one), or 0.
unsigned long long capture_id(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  if (hipStreamGetCaptureInfo(stream, &st, &id) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return st == hipStreamCaptureStatusActive ? id : 0;
}

// Note when the graph that `stream` is being captured into is no more (the
// callback may come on any thread and calls no HIP function).
std::shared_ptr<std::atomic<bool>> watch_graph(hipStream_t stream) {
  using Mark = std::shared_ptr<std::atomic<bool>>;
  Mark mark = std::make_shared<std::atomic<bool>>(false);
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  hipGraph_t graph = nullptr;
  const hipGraphNode_t* deps = nullptr;
  size_t n_deps = 0;
  hipUserObject_t object = nullptr;
  Mark* held = new Mark(mark);
  auto tell = [](void* p) {
    Mark* m = static_cast<Mark*>(p);
    (*m)->store(true);
    delete m;
  };
  if (hipStreamGetCaptureInfo_v2(stream, &st, &id, &graph, &deps, &n_deps) != hipSuccess ||
      !graph ||
      hipUserObjectCreate(&object, held, tell, 1, hipUserObjectNoDestructorSync) != hipSuccess) {
    (void)hipGetLastError();
    delete held;
    return mark;  // never told: the buffer stays until ccc_release_workspace
  }
  if (hipGraphRetainUserObject(graph, object, 1, hipGraphUserObjectMove) != hipSuccess) {
    (void)hipGetLastError();
    mark = std::make_shared<std::atomic<bool>>(false);  // likewise; the object has the old one
    (void)hipUserObjectRelease(object, 1);
  }
  return mark;
}

// hipMalloc that is also allowed while a stream of this thread is captured.
void* allocate(size_t bytes, bool capture) {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (capture && hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  void* p = nullptr;
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    p = nullptr;
  }
  if (capture) (void)hipThreadExchangeStreamCaptureMode(&mode);
  return p;
}

bool is_gone(const Workspace& w) { return w.gone && w.gone->load(); }

// Free the buffers of the workspaces on `dev` that `which` picks; the device has
// been waited for.
template <typename Which>
void free_buffers(int dev, Which which) {
  for (auto* list : {&g_ws, &g_retired})
    for (Workspace& w : *list) {
      if (w.dev != dev || !which(w)) continue;
      if (w.ptr) (void)hipFree(w.ptr);
      if (w.ops) (void)hipFree(w.ops);
      w.ptr = w.ops = nullptr;
      w.bytes = w.ops_bytes = 0;
    }
}

bool wait_for_device() {
  if (hipDeviceSynchronize() == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

// Room for `bytes` of operands besides those held on the device, `own` of which
// the caller would give back.
bool room_for_operands(int dev, size_t bytes, size_t own, bool capture) {
  int64_t held = (int64_t)bytes - (int64_t)own;
  for (auto* list : {&g_ws, &g_retired})
    for (const Workspace& w : *list)
      if (w.dev == dev) held += (int64_t)w.ops_bytes;
  if (auto it = g_batch_operands.find(dev); it != g_batch_operands.end()) held += it->second;
  if (held > operand_limit()) return false;
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (capture && hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  size_t avail = 0, total = 0;
  const bool known = hipMemGetInfo(&avail, &total) == hipSuccess;
  if (!known) (void)hipGetLastError();
  if (capture) (void)hipThreadExchangeStreamCaptureMode(&mode);
  return known && bytes <= avail && bytes <= (avail + own) / 2;
}

// At least `bytes` of operand space in w, or not: never at another workspace's
// cost, and where there is no room without waiting for anything.
bool operand_space(Workspace& w, size_t bytes) {
  if ((int64_t)bytes > operand_limit()) return false;
  if (w.ops_bytes >= bytes) return true;
  const bool capture = w.capture != 0;
  const size_t own = capture ? 0 : w.ops_bytes;  // a graph keeps what it outgrew
  if (!room_for_operands(w.dev, bytes, own, capture)) return false;
  if (w.ops && !capture && !wait_for_device()) return false;  // its work may still be going on
  void* p = allocate(bytes, capture);
  if (!p) return false;
  if (w.ops && capture) {
    Workspace old = w;
    old.ptr = nullptr;
    old.bytes = 0;
    g_retired.push_back(old);
  } else if (w.ops) {
    (void)hipFree(w.ops);
  }
  w.ops = p;
  w.ops_bytes = bytes;
  return true;
}

}  // namespace

// The workspace of `stream` on the current device, grown on demand: at least
// `bytes` at *out, and with op_bytes > 0 as many at *ops, or null there when
// the operands have no room.  `lock` is held until the caller has enqueued its
// work.
int workspace(size_t bytes, size_t op_bytes, hipStream_t stream,
              std::unique_lock<std::mutex>& lock, char** out, char** ops) try {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return CCC_ERR_HIP;
  const size_t thread =
      stream == hipStreamPerThread ? std::hash<std::thread::id>()(std::this_thread::get_id()) : 0;
  const unsigned long long capture = capture_id(stream);
  lock = std::unique_lock<std::mutex>(g_mu);
  auto gone_here = [&](const Workspace& w) { return w.dev == dev && is_gone(w); };
  size_t gone = 0, gone_bytes = 0;
  for (auto* list : {&g_ws, &g_retired})
    for (const Workspace& w : *list)
      if (gone_here(w)) {
        ++gone;
        gone_bytes += w.bytes + w.ops_bytes;
      }
  if (!capture && (gone > kMaxGone || gone_bytes > kMaxGoneBytes) && wait_for_device()) {
    free_buffers(dev, is_gone);
    for (auto* list : {&g_ws, &g_retired})
      list->erase(std::remove_if(list->begin(), list->end(),
                                 [&](const Workspace& w) { return gone_here(w) && !w.ptr && !w.ops; }),
                  list->end());
  }
  size_t at = 0;
  while (at < g_ws.size() && !(g_ws[at].dev == dev && g_ws[at].stream == stream &&
                               g_ws[at].thread == thread && g_ws[at].capture == capture))
    ++at;
  if (at == g_ws.size()) {
    std::vector<uint64_t> used;  // last uses of the other streams'
    for (const Workspace& w : g_ws)
      if (w.dev == dev && !w.capture) used.push_back(w.last_use);
    if (used.size() >= kMaxWorkspaces && !capture && wait_for_device()) {
      std::nth_element(used.begin(), used.begin() + used.size() / 2, used.end());
      const uint64_t median = used[used.size() / 2];
      auto old = [&](const Workspace& w) {
        return w.dev == dev && !w.capture && w.last_use < median;
      };
      free_buffers(dev, old);
      g_ws.erase(std::remove_if(g_ws.begin(), g_ws.end(), old), g_ws.end());
    }
    at = g_ws.size();
    g_ws.push_back(Workspace{});
    g_ws[at].dev = dev;
    g_ws[at].stream = stream;
    g_ws[at].thread = thread;
    g_ws[at].capture = capture;
    if (capture) g_ws[at].gone = watch_graph(stream);
  }
  Workspace& w = g_ws[at];
  if (w.bytes < bytes) {
    if (w.ptr && capture) {
      Workspace old = w;
      old.ops = nullptr;
      old.ops_bytes = 0;
      g_retired.push_back(old);
    } else if (w.ptr) {
      // the old buffer may still be in use by enqueued work
      if (hipDeviceSynchronize() != hipSuccess) return CCC_ERR_HIP;
      (void)hipFree(w.ptr);
    }
    w.ptr = nullptr;
    w.bytes = 0;
    const size_t want = bytes < (1u << 20) ? (1u << 20) : bytes;
    w.ptr = allocate(want, capture);
    if (!w.ptr && !capture && wait_for_device()) {  // whatever no graph holds makes room
      free_buffers(dev, [](const Workspace& x) { return !x.capture || is_gone(x); });
      w.ptr = allocate(want, false);
    }
    if (!w.ptr) return CCC_ERR_NOMEM;
    w.bytes = want;
  }
  w.last_use = ++g_clock;
  *out = static_cast<char*>(w.ptr);
  if (ops) *ops = op_bytes > 0 && operand_space(w, op_bytes) ? static_cast<char*>(w.ops) : nullptr;
  return CCC_OK;
} catch (const std::bad_alloc&) {  // of the host's own lists
  return CCC_ERR_NOMEM;
}

bool batch_operands_fit(int dev, size_t bytes) {
  std::lock_guard<std::mutex> lk(g_mu);
  return room_for_operands(dev, bytes, 0, false);
}
void hold_batch_operands(int dev, int64_t bytes) {
  std::lock_guard<std::mutex> lk(g_mu);
  g_batch_operands[dev] += bytes;
}

static int run_pair2(const Pair2Args& a, int path, hipStream_t stream) {
  hipError_t e = path == CCC_PATH_POPCOUNT ? launch_pop2(a, stream) : launch_mfma2(a, stream);
  return e == hipSuccess ? CCC_OK : CCC_ERR_HIP;
}

}  // namespace ccc

extern "C" {

ccc_opts ccc_default_opts(void) {
  ccc_opts o;
  o.path = CCC_PATH_AUTO;
  o.gamma = 2.0 / 3.0;
  o.flags = 0;
  o.operands = CCC_OPERANDS_AUTO;
  return o;
}

int ccc_version(void) { return 200; }

int ccc_mfma_operands(int64_t n_f) {
  if (n_f < 0) return CCC_ERR_ARG;
  return n_f <= ccc::kF4MaxFields ? CCC_OPERANDS_FP4 : CCC_OPERANDS_INT8;
}

const char* ccc_status_string(int status) {
  switch (status) {
    case CCC_OK: return "ok";
    case CCC_ERR_ARG: return "invalid argument";
    case CCC_ERR_RANGE: return "a table entry could exceed the int32 range";
    case CCC_ERR_ALIGN: return "pointer not 16-byte aligned or row stride not a multiple of 16";
    case CCC_ERR_HIP: return "HIP call or kernel launch failed";
    case CCC_ERR_NOMEM: return "workspace allocation failed";
    case CCC_ERR_UNSUPPORTED: return "unsupported";
    default: return "unknown status";
  }
}

}  // extern "C"

namespace {

// All 2-way variants: dense rows [i_begin, i_end) (tables/ccc) or selection.
int two_way(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, int64_t i_begin,
            int64_t i_end, int32_t* tables, double* ccc, const ccc_selection* sel,
            double threshold, int32_t* counts, const ccc_opts* opts, hipStream_t stream) {
  ccc_opts o;
  int st = resolve_opts(opts, &o);
  if (st) return st;
  if (o.flags != 0) return CCC_ERR_ARG;
  if ((st = check_input(v, n_v, n_f, ld))) return st;
  if (!fields_in_range(n_f, 4)) return CCC_ERR_RANGE;
  const int f4 = o.path == CCC_PATH_POPCOUNT ? 0 : use_fp4(o, n_f);
  if (f4 < 0) return f4;
  if (i_begin < 0 || i_end < i_begin || i_end > n_v) return CCC_ERR_ARG;
  if (sel) {
    if (!sel->index || !sel->ccc || !sel->count || sel->cap < 0) return CCC_ERR_ARG;
    if (!isfinite(threshold)) return CCC_ERR_ARG;
    if (!aligned16(sel->index) || !aligned16(sel->ccc) || !aligned16(sel->tables) ||
        !aligned16(sel->count))
      return CCC_ERR_ALIGN;
  } else if ((i_end < n_v - 1 ? i_end : n_v - 1) > i_begin && !tables && !ccc) {
    return CCC_ERR_ARG;  // the range holds pairs but there is nowhere to put them
  }
  if (!aligned16(tables) || !aligned16(ccc) || !aligned16(counts)) return CCC_ERR_ALIGN;
  if (n_v == 0) return CCC_OK;
  unsigned long long* zero = sel ? sel->count : nullptr;
  const int64_t row_end = i_end < n_v - 1 ? i_end : n_v - 1;  // the last row has no pair
  if (row_end <= i_begin && !counts && !zero) return CCC_OK;  // nothing to compute or write
  std::unique_lock<std::mutex> lock;
  if (n_v == 1) {
    if (!counts && !zero) return CCC_OK;
    if (!counts) {  // only the selection counter to clear
      char* ws = nullptr;
      if ((st = ccc::workspace(16, 0, stream, lock, &ws, nullptr))) return st;
      counts = reinterpret_cast<int32_t*>(ws);
    }
    return ccc::launch_count1_zero(v, ld, n_v, n_f, counts, 0, zero, stream) == hipSuccess
               ? CCC_OK
               : CCC_ERR_HIP;
  }
  ccc::Pair2Args a{};
  a.va = v; a.lda = ld; a.n_a = n_v;
  a.vb = v; a.ldb = ld; a.n_b = n_v;
  a.n_f = n_f;
  a.f4 = f4;
  a.tri = 1;
  a.accumulate = 0;
  a.tables = tables;
  a.ccc = ccc;
  a.gamma = o.gamma;
  a.row_begin = i_begin;
  a.row_end = row_end;
  a.p_base = i_begin * n_v - i_begin * (i_begin + 1) / 2;  // p(i_begin, i_begin + 1)
  a.sel = sel ? ccc::Select{sel->count, sel->cap, threshold, sel->index, sel->ccc, sel->tables}
              : ccc::Select{nullptr, 0, 0.0, nullptr, nullptr, nullptr};
  // workspace: the MFMA path's complete-data flag, the counts (unless the
  // caller's), and on fp4 the operands and the partial sums of split tiles
  const bool have_pairs = row_end > i_begin;
  const size_t cnt_bytes = counts ? 0 : round256((size_t)n_v * 16);
  const size_t head = 256 + cnt_bytes;
  size_t op_bytes = 0, part_bytes = 0;
  const int64_t first = ccc::operand_first(i_begin);  // earlier rows are in no pair of the range
  if (f4 && have_pairs && ccc::operands_serve(a)) {
    a.steps = ccc::operand_steps(n_f);
    op_bytes = (size_t)ccc::operand_bytes(n_v - 16 * first, n_f);
    a.part_bytes = ccc::mfma2_part_bytes(a);
    // the pre-pass is done with its part when the tiles write theirs
    const size_t pre_bytes = ccc::operand_part_bytes(n_v, n_f);
    part_bytes = pre_bytes > a.part_bytes ? pre_bytes : a.part_bytes;
  }
  char *wsb = nullptr, *z = nullptr;
  if ((st = ccc::workspace(head, op_bytes + part_bytes, stream, lock, &wsb, &z))) return st;
  int32_t* cnt = counts ? counts : reinterpret_cast<int32_t*>(wsb + 256);
  a.counts_a = a.counts_b = a.chunk_a = a.chunk_b = cnt;
  a.flag = reinterpret_cast<unsigned long long*>(wsb);
  a.id = g_call++;
  if (z) {
    // block 0's address, were it laid out
    a.za = a.zb = reinterpret_cast<const void*>(reinterpret_cast<uintptr_t>(z) -
                                                (uintptr_t)(first * a.steps * 1024));
    a.part = z + op_bytes;
    ccc::OperandJob job{};
    job.set[0] = ccc::OperandSet{v, ld, n_v, (uint32_t)ccc::operand_blocks(n_v), (uint32_t)first, z,
                                 cnt, nullptr};
    job.n_f = n_f;
    job.steps = a.steps;
    job.zero = zero;
    job.flag = a.flag;
    job.id = a.id;
    job.shares = ccc::operand_shares(n_v, n_f);
    job.part = static_cast<int2*>(a.part);
    if (ccc::launch_operands(job, stream) != hipSuccess) return CCC_ERR_HIP;
  } else if (ccc::launch_count1_zero(v, ld, n_v, n_f, cnt, 0, zero, stream) != hipSuccess) {
    return CCC_ERR_HIP;
  }
  if (!have_pairs) return CCC_OK;
  return ccc::run_pair2(a, o.path, stream);
}

int64_t choose3(int64_t n) { return n < 3 ? 0 : n * (n - 1) / 2 * (n - 2) / 3; }
int64_t choose2(int64_t n) { return n < 2 ? 0 : n * (n - 1) / 2; }

// Scratch of ccc_3way_noalloc: a fixed device array, one copy per device,
// held until the process ends.  Host code never uses its name as an address:
// the device address of each device's copy is looked up once (with that
// device current) and kept in g_scratch.
static __device__ __align__(256) unsigned char scratch[CCC_NOALLOC_SCRATCH_BYTES];

std::mutex g_scratch_mu;
std::vector<void*> g_scratch;  // indexed by device ordinal; null until looked up

int noalloc_scratch(char** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return CCC_ERR_HIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if ((int)g_scratch.size() <= dev) g_scratch.resize(dev + 1, nullptr);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return CCC_ERR_HIP;
    }
    g_scratch[dev] = p;
  }
  *out = static_cast<char*>(g_scratch[dev]);
  return CCC_OK;
}

// The no-allocation form of a call: its scratch is the fixed array above
// (`bytes` of it) instead of the library workspace.
struct FixedScratch {
  size_t bytes;
};

// All 3-way variants: dense first-index rows [i_begin, i_end) or selection.
// With `fixed`, the scratch comes from there instead of the workspace: the
// call returns CCC_ERR_RANGE past the documented bound on n_v, and
// leaves the Gram matrix out (every unit then takes the general form, same
// results) when it does not fit beside them.
int three_way(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, int64_t i_begin,
              int64_t i_end, int32_t* tables, double* ccc, const ccc_selection* sel,
              double threshold, int32_t* counts, const ccc_opts* opts, hipStream_t stream,
              const FixedScratch* fixed = nullptr) {
  ccc_opts o;
  int st = resolve_opts(opts, &o);
  if (st) return st;
  if (o.flags != 0) return CCC_ERR_ARG;
  if ((st = check_input(v, n_v, n_f, ld))) return st;
  if (!fields_in_range(n_f, 8)) return CCC_ERR_RANGE;
  const int f4 = o.path == CCC_PATH_POPCOUNT ? 0 : use_fp4(o, n_f);
  if (f4 < 0) return f4;
  if (i_begin < 0 || i_end < i_begin || i_end > n_v) return CCC_ERR_ARG;
  if (sel) {
    if (!sel->index || !sel->ccc || !sel->count || sel->cap < 0) return CCC_ERR_ARG;
    if (!isfinite(threshold)) return CCC_ERR_ARG;
    if (!aligned16(sel->index) || !aligned16(sel->ccc) || !aligned16(sel->tables) ||
        !aligned16(sel->count))
      return CCC_ERR_ALIGN;
  } else if ((i_end < n_v - 2 ? i_end : n_v - 2) > i_begin && !tables && !ccc) {
    return CCC_ERR_ARG;  // the range holds triples but there is nowhere to put them
  }
  if (!aligned16(tables) || !aligned16(ccc) || !aligned16(counts)) return CCC_ERR_ALIGN;
  if (n_v > 2642245) return CCC_ERR_ARG;  // C(n_v,3) * 8 must fit int64 indexing
  if (n_v == 0) return CCC_OK;
  unsigned long long* zero = sel ? sel->count : nullptr;
  const int64_t row_end = i_end < n_v - 2 ? i_end : n_v - 2;  // first index below n_v - 2
  if (row_end <= i_begin && !counts && !zero) return CCC_OK;  // nothing to compute or write
  // scratch: the complete-data flag, the counts (unless the caller's), then
  // (MFMA path) the rho(1) Gram matrix of rows [g0, n_v) used by complete-data
  // units; g0 is i_begin rounded down to the unit tile
  const size_t cnt_bytes = counts ? 0 : round256((size_t)n_v * 16);
  const size_t head_bytes = 256 + cnt_bytes;
  const int64_t g0 = i_begin / ccc::kUnitTile * ccc::kUnitTile, ng = n_v - g0;
  bool use_gram = o.path != CCC_PATH_POPCOUNT && ng <= kGramMaxRows && i_begin < row_end;
  // Small fp4 calls take the general kernel whatever their rows: the Gram
  // matrix and the complete-data kernel's few, longer workgroups cost more than
  // its eight planes while its units make one turn of the chip, and in two
  // turns while the fields are not long (us, complete data, complete-data form /
  // general: 60 x 2000 83 / 34, 120 x 10000 150 / 67, 180 x 200000, 430 units,
  // 1484 / 1207; 200 x 10000, 630 units, 185 / 135, 200 x 100000 884 / 917; 228 x
  // 20000, 904 units, 286 / 276, 228 x 40000 430 / 492; 260 x 1000, 1257 units,
  // 121 / 91, but 260 x 10000 187 / 204 and 260 x 50000 476 / 721).
  if (f4 && use_gram) {
    const int64_t units =
        ccc::grid_unit_count(ccc::unit_grid(n_v, ccc::kRunTile, i_begin, row_end, 4));
    if (units <= 512 || (units <= 1024 && units * n_f <= 20000000) ||
        (units < 2048 && n_f <= 2048))
      use_gram = false;
  }
  if (fixed) {
    // the bound of the documented interface: tables of unit offsets (8 bytes
    // per tile pair of three unit grids) that the kernels no longer need
    const ccc::UnitGrid u64 = ccc::unit_grid(n_v, ccc::kUnitTile, i_begin, row_end);
    const ccc::UnitGrid u32 = ccc::unit_grid(n_v, ccc::kRunTile, i_begin, row_end);
    const size_t bound = 2 * round256((size_t)(ccc::grid_pairs(u64) + 1) * 8) +
                         round256((size_t)(ccc::grid_pairs(u32) + 1) * 8) + head_bytes;
    if (bound > fixed->bytes) return CCC_ERR_RANGE;
    if (use_gram && (size_t)ng * (size_t)ng * 4 > fixed->bytes - bound) use_gram = false;
  }
  const size_t gram_bytes = use_gram ? (size_t)ng * (size_t)ng * 4 : 0;
  char* wsb = nullptr;
  std::unique_lock<std::mutex> lock;
  if ((st = fixed ? noalloc_scratch(&wsb)
                  : ccc::workspace(head_bytes + gram_bytes, 0, stream, lock, &wsb, nullptr)))
    return st;
  int32_t* cnt = counts ? counts : reinterpret_cast<int32_t*>(wsb + 256);
  ccc::Triple3Args a{};
  // the complete-data kernel (fp4 operands, with the Gram matrix)
  a.flag = use_gram && f4 && n_f > 0 ? reinterpret_cast<unsigned long long*>(wsb) : nullptr;
  a.id = g_call++;
  if (ccc::launch_count1_zero(v, ld, n_v, n_f, cnt, 0, zero, stream, a.flag, a.id, g0) !=
      hipSuccess)
    return CCC_ERR_HIP;
  if (n_v < 3 || row_end <= i_begin) return CCC_OK;
  a.v = v; a.ld = ld; a.n = n_v; a.n_f = n_f;
  a.f4 = f4;
  a.tables = tables;
  a.ccc = ccc;
  a.counts = cnt;
  a.gamma = o.gamma;
  a.i_begin = i_begin;
  a.i_end = row_end;
  a.t_base = choose3(n_v) - choose3(n_v - i_begin);  // T(i_begin, i_begin+1, i_begin+2)
  a.sel = sel ? ccc::Select{sel->count, sel->cap, threshold, sel->index, sel->ccc, sel->tables}
              : ccc::Select{nullptr, 0, 0.0, nullptr, nullptr, nullptr};
  a.gram = use_gram ? reinterpret_cast<int32_t*>(wsb + head_bytes) : nullptr;
  a.g0 = g0;
  a.ng = use_gram ? ng : 0;
  hipError_t e = o.path == CCC_PATH_POPCOUNT ? ccc::launch_pop3(a, stream)
                                             : ccc::launch_mfma3(a, stream);
  return e == hipSuccess ? CCC_OK : CCC_ERR_HIP;
}

}  // namespace

extern "C" {

int ccc_2way(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, int32_t* tables,
             double* ccc, int32_t* counts, const ccc_opts* opts, hipStream_t stream) {
  return two_way(v, n_v, n_f, ld, 0, n_v < 0 ? 0 : n_v, tables, ccc, nullptr, 0.0, counts, opts,
                 stream);
}

int ccc_2way_rows(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, int64_t i_begin,
                  int64_t i_end, int32_t* tables, double* ccc, int32_t* counts,
                  const ccc_opts* opts, hipStream_t stream) {
  return two_way(v, n_v, n_f, ld, i_begin, i_end, tables, ccc, nullptr, 0.0, counts, opts,
                 stream);
}

int ccc_2way_select(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, double threshold,
                    const ccc_selection* out, int32_t* counts, const ccc_opts* opts,
                    hipStream_t stream) {
  if (!out) return CCC_ERR_ARG;
  return two_way(v, n_v, n_f, ld, 0, n_v < 0 ? 0 : n_v, nullptr, nullptr, out, threshold,
                 counts, opts, stream);
}

int ccc_3way_rows(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, int64_t i_begin,
                  int64_t i_end, int32_t* tables, double* ccc, int32_t* counts,
                  const ccc_opts* opts, hipStream_t stream) {
  return three_way(v, n_v, n_f, ld, i_begin, i_end, tables, ccc, nullptr, 0.0, counts, opts,
                   stream);
}

int ccc_3way_select(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, double threshold,
                    const ccc_selection* out, int32_t* counts, const ccc_opts* opts,
                    hipStream_t stream) {
  if (!out) return CCC_ERR_ARG;
  return three_way(v, n_v, n_f, ld, 0, n_v < 0 ? 0 : n_v, nullptr, nullptr, out, threshold,
                   counts, opts, stream);
}

int ccc_3way(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, int32_t* tables,
             double* ccc, int32_t* counts, const ccc_opts* opts, hipStream_t stream) {
  return three_way(v, n_v, n_f, ld, 0, n_v < 0 ? 0 : n_v, tables, ccc, nullptr, 0.0, counts,
                   opts, stream);
}

int ccc_2way_block(const uint8_t* va, int64_t n_a, int64_t lda, const uint8_t* vb, int64_t n_b,
                   int64_t ldb, int64_t n_f, int32_t* tables, int32_t* counts_a,
                   int32_t* counts_b, double* ccc, const ccc_opts* opts, hipStream_t stream) {
  ccc_opts o;
  int st = resolve_opts(opts, &o);
  if (st) return st;
  if ((st = check_input(va, n_a, n_f, lda))) return st;
  if ((st = check_input(vb, n_b, n_f, ldb))) return st;
  if (!fields_in_range(n_f, 4)) return CCC_ERR_RANGE;
  const int f4 = o.path == CCC_PATH_POPCOUNT ? 0 : use_fp4(o, n_f);
  if (f4 < 0) return f4;
  const bool acc = (o.flags & CCC_ACCUMULATE) != 0, fin = (o.flags & CCC_FINALIZE) != 0;
  if (n_a > 0 && n_b > 0) {
    if (!tables || !counts_a || !counts_b) return CCC_ERR_ARG;
    if (fin && !ccc) return CCC_ERR_ARG;
  }
  if (!aligned16(tables) || !aligned16(ccc) || !aligned16(counts_a) || !aligned16(counts_b))
    return CCC_ERR_ALIGN;
  if (n_a == 0 || n_b == 0) return CCC_OK;
  ccc::Pair2Args a{};
  a.va = va; a.lda = lda; a.n_a = n_a;
  a.vb = vb; a.ldb = ldb; a.n_b = n_b;
  a.n_f = n_f;
  a.f4 = f4;
  a.tri = 0;
  a.accumulate = acc ? 1 : 0;
  a.tables = tables;
  a.ccc = fin ? ccc : nullptr;
  a.counts_a = counts_a;
  a.counts_b = counts_b;
  a.gamma = o.gamma;
  a.row_begin = 0;
  a.row_end = n_a;
  a.p_base = 0;
  a.sel = ccc::Select{nullptr, 0, 0.0, nullptr, nullptr, nullptr};
  // workspace: the MFMA path's complete-data flag, an accumulating call's own
  // chunk counts, and on fp4 the operands of both sides and the partial sums
  // of split tiles
  const size_t cnt_bytes = acc ? round256((size_t)(n_a + n_b) * 16) : 0, head = 256 + cnt_bytes;
  const size_t op_a = (size_t)ccc::operand_bytes(n_a, n_f), op_b = (size_t)ccc::operand_bytes(n_b, n_f);
  std::unique_lock<std::mutex> lock;
  size_t op_bytes = 0;
  if (f4 && ccc::operands_serve(a)) {
    a.steps = ccc::operand_steps(n_f);
    a.part_bytes = ccc::mfma2_part_bytes(a);
    op_bytes = op_a + op_b + a.part_bytes;
  }
  char *wsb = nullptr, *z = nullptr;
  if ((st = ccc::workspace(head, op_bytes, stream, lock, &wsb, &z))) return st;
  int32_t* chunk_a = acc ? reinterpret_cast<int32_t*>(wsb + 256) : counts_a;
  int32_t* chunk_b = acc ? chunk_a + 4 * n_a : counts_b;
  a.chunk_a = chunk_a;
  a.chunk_b = chunk_b;
  a.flag = acc ? nullptr : reinterpret_cast<unsigned long long*>(wsb);
  a.id = g_call++;
  if (z) {
    a.za = z;
    a.zb = z + op_a;
    a.part = z + op_a + op_b;
    ccc::OperandJob job{};
    job.set[0] = ccc::OperandSet{va, lda, n_a, (uint32_t)ccc::operand_blocks(n_a), 0, z, counts_a,
                                 acc ? chunk_a : nullptr};
    job.set[1] = ccc::OperandSet{vb, ldb, n_b, (uint32_t)ccc::operand_blocks(n_b), 0, z + op_a,
                                 counts_b, acc ? chunk_b : nullptr};
    job.n_f = n_f;
    job.steps = a.steps;
    job.accumulate = acc ? 1 : 0;
    job.flag = a.flag;
    job.id = a.id;
    // Counts that share entries (both sides rows of one set, say) are written
    // or added to one side after the other, as by the passes over packed rows.
    const bool shared = counts_a < counts_b + 4 * n_b && counts_b < counts_a + 4 * n_a;
    const ccc::OperandSet second = job.set[1];
    if (shared) job.set[1] = ccc::OperandSet{};
    if (ccc::launch_operands(job, stream) != hipSuccess) return CCC_ERR_HIP;
    if (shared) {
      job.set[0] = second;
      if (ccc::launch_operands(job, stream) != hipSuccess) return CCC_ERR_HIP;
    }
  } else {
    if (acc && (ccc::launch_count1(va, lda, n_a, n_f, chunk_a, 0, stream) != hipSuccess ||
                ccc::launch_count1(vb, ldb, n_b, n_f, chunk_b, 0, stream) != hipSuccess))
      return CCC_ERR_HIP;
    if (ccc::launch_count1(va, lda, n_a, n_f, counts_a, acc, stream) != hipSuccess ||
        ccc::launch_count1(vb, ldb, n_b, n_f, counts_b, acc, stream) != hipSuccess)
      return CCC_ERR_HIP;
  }
  return ccc::run_pair2(a, o.path, stream);
}

int ccc_2way_multi(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, int s,
                   int32_t* tables, double* ccc, int32_t* counts, const ccc_opts* opts,
                   hipStream_t stream) {
  ccc_opts o;
  int st = resolve_opts(opts, &o);
  if (st) return st;
  if (o.flags != 0) return CCC_ERR_ARG;
  if (o.path == CCC_PATH_POPCOUNT) return CCC_ERR_UNSUPPORTED;
  if (s < 2 || s > 4) return CCC_ERR_ARG;
  if (n_v < 0 || n_f < 0 || ld < 0 || n_v > kInt32Max) return CCC_ERR_ARG;
  if (ld % 16 != 0) return CCC_ERR_ALIGN;
  if (ld > kMaxLd) return CCC_ERR_RANGE;
  if (ld < n_f) return CCC_ERR_ARG;
  if (n_v > 0 && !v) return CCC_ERR_ARG;
  if (!aligned16(v) || !aligned16(tables) || !aligned16(ccc) || !aligned16(counts))
    return CCC_ERR_ALIGN;
  if (!fields_in_range(n_f, 4)) return CCC_ERR_RANGE;
  const int f4 = use_fp4(o, n_f);
  if (f4 < 0) return f4;
  if (n_v >= 2 && !tables && !ccc) return CCC_ERR_ARG;
  if (n_v == 0 || (n_v == 1 && !counts)) return CCC_OK;
  // workspace: the counts (unless the caller's) and on fp4 the operands
  std::unique_lock<std::mutex> lock;
  const size_t cnt_bytes = counts ? 0 : round256((size_t)n_v * 32);
  const size_t op_bytes = f4 && n_v >= 2 && n_f > 0 ? ccc::multi_operand_bytes(n_v, n_f, s) : 0;
  char *ws = nullptr, *z = nullptr;
  if ((cnt_bytes || op_bytes) &&
      (st = ccc::workspace(cnt_bytes, op_bytes, stream, lock, &ws, &z)))
    return st;
  int32_t* cnt = counts ? counts : reinterpret_cast<int32_t*>(ws);
  const hipError_t e =
      z ? ccc::launch_multi_operands(v, ld, n_v, n_f, s, cnt, z, stream)
        : ccc::launch_multi_count(v, ld, n_v, n_f, s, cnt, stream);
  if (e != hipSuccess) return CCC_ERR_HIP;
  if (n_v < 2) return CCC_OK;
  return ccc::launch_multi2(v, ld, n_v, n_f, s, tables, ccc, cnt, o.gamma, f4, z, stream) ==
                 hipSuccess
             ? CCC_OK
             : CCC_ERR_HIP;
}

int ccc_2way_many(const ccc_problem* probs, int n_probs, const ccc_opts* opts,
                  hipStream_t stream) {
  ccc_opts o;
  int st = resolve_opts(opts, &o);
  if (st) return st;
  if (o.flags != 0) return CCC_ERR_ARG;
  if (n_probs < 0 || (n_probs > 0 && !probs)) return CCC_ERR_ARG;
  int64_t nf_max = 0;
  for (int p = 0; p < n_probs; ++p) {
    const ccc_problem& q = probs[p];
    if ((st = check_input(q.v, q.n_v, q.n_f, q.ld))) return st;
    if (!fields_in_range(q.n_f, 4)) return CCC_ERR_RANGE;
    if (q.n_f > nf_max) nf_max = q.n_f;
    if (q.n_v >= 2 && !q.tables && !q.ccc) return CCC_ERR_ARG;
    if (!aligned16(q.tables) || !aligned16(q.ccc) || !aligned16(q.counts)) return CCC_ERR_ALIGN;
  }
  const int f4 = o.path == CCC_PATH_POPCOUNT ? 0 : use_fp4(o, nf_max);
  if (f4 < 0) return f4;
  if (n_probs == 0) return CCC_OK;
  return ccc::run_many(probs, n_probs, o, f4 != 0, stream);
}

int ccc_3way_noalloc(const uint8_t* v, int64_t n_v, int64_t n_f, int64_t ld, int32_t* tables,
                     double* ccc, int32_t* counts, const ccc_opts* opts, hipStream_t stream) {
  const FixedScratch fs{CCC_NOALLOC_SCRATCH_BYTES};
  return three_way(v, n_v, n_f, ld, 0, n_v < 0 ? 0 : n_v, tables, ccc, nullptr, 0.0, counts,
                   opts, stream, &fs);
}

void ccc_release_workspace(void) {
  ccc::release_many_cache();
  std::lock_guard<std::mutex> lk(g_mu);
  int cur = 0;
  bool have_cur = hipGetDevice(&cur) == hipSuccess;
  for (auto* list : {&g_ws, &g_retired}) {
    for (const Workspace& w : *list) {
      if (!w.ptr && !w.ops) continue;
      if (hipSetDevice(w.dev) == hipSuccess) {
        (void)hipDeviceSynchronize();
        (void)hipFree(w.ptr);
        (void)hipFree(w.ops);
      }
    }
    list->clear();
  }
  if (have_cur) (void)hipSetDevice(cur);
}

}  // extern "C"
