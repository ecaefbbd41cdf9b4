// C ABI of the library: argument checks (host only, before any HIP call),
// context state (stencil tables, descriptor/work-list caches, captured
// graphs, tuning choices) and dispatch to the kernels.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <memory>
#include <string>
#include <unordered_map>
#include <vector>

#include "kernels.h"
#include "m2l_mfma.h"
#include "stencil_pairs.h"

using namespace fmm;

// Device memory of fmm_m2l_noalloc: descriptors, work counter and work list of
// one call, at most FMM_NOALLOC_MAX_SUBGRIDS sub-grids. One copy per device,
// held until the process ends; every call on a device shares it. Host code
// never passes this name to a kernel or a copy: fmm_create looks up each
// device's address of it (fmm_ctx::noalloc_dev) and that address is used.
constexpr size_t kNoAllocDescBytes = sizeof(fmm_subgrid) * FMM_NOALLOC_MAX_SUBGRIDS;
constexpr size_t kNoAllocCounterOff = (kNoAllocDescBytes + 255) / 256 * 256;   // inside every call's upload
constexpr size_t kNoAllocWorkOff = kNoAllocCounterOff + 256;
constexpr size_t kNoAllocItems = (size_t)max_parts(FMM_NOALLOC_MAX_SUBGRIDS);   // parts of the sub-grids
constexpr size_t kNoAllocBytes = kNoAllocWorkOff + sizeof(WorkItem) * kNoAllocItems;
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {

thread_local std::string g_create_error;

const char* kStatusStrings[] = {"FMM_OK", "FMM_EINVAL: invalid argument",
                                "FMM_ENOMEM: out of memory", "FMM_EHIP: HIP runtime error",
                                "FMM_EUNSUPPORTED: unsupported request"};

uint64_t fnv1a(const void* data, size_t n, uint64_t h = 1469598103934665603ull) {
  const unsigned char* p = static_cast<const unsigned char*>(data);
  for (size_t i = 0; i < n; ++i) {
    h ^= p[i];
    h *= 1099511628211ull;
  }
  return h;
}

}  // namespace

// Work lists of one form's forward or adjoint calls on a descriptor set, made by
// the first of them (P2M and evaluation need none): in the set's allocation, or for
// large sets, unless that call is the set's first, in one of their own.
struct CallLists {
  bool made = false;
  void* dev = nullptr;            // (own device allocation and pinned host copy, if any)
  void* pinned = nullptr;
  WorkList whole;                 // sub-grids, longest first; a counter that the launches leave at zero, and
                                  // after it one that the per-wave launches reset
  WorkList cut;                   // their parts (forward) or rounds (adjoint), where planned or asked for
};
// the lists a call needs
constexpr int need_forward(bool harmonic) { return harmonic ? 1 : 0; }
constexpr int need_adjoint(bool harmonic) { return harmonic ? 3 : 2; }
constexpr int kNeedNone = -1;
constexpr int64_t kRoomSubgrids = 1024;   // sets of up to so many keep room for all lists (0.5 MB)

// Descriptor set uploaded to the device, plus everything derived from it.
struct DescEntry {
  std::vector<fmm_subgrid> host;
  uint64_t hash = 0;
  uint64_t id = 0;                // unique per upload (keys this set's graphs)
  uint64_t last_use = 0;
  void* dev = nullptr;            // one device allocation: descriptors, id lists, the first call's work lists
  void* pinned = nullptr;         // pinned host copy of the same bytes
  size_t bytes = 0;
  DevDesc* d_desc = nullptr;
  int* d_ids[kMaxP + 1] = {};     // reference kernels: sub-grids per order
  int count[kMaxP + 1] = {};
  CallLists lists[4];             // by need
  size_t room[4] = {};            // their places in the allocation, if kept there
  StreamPlan plan[2];             // made with the lists
  AdjointPlan adjoint_plan[2];
  bool part_even = true;          // every part_off even: particle blocks 16-byte aligned
  int tuned[4] = {-1, -1, -1, -1};   // autotuned configuration per precision
  int tuned_parts[4] = {-1, -1, -1, -1};   // and whether it runs parts of sub-grids (-1: as planned)
  // FMM_EXACT_SLICE: the sub-grids' slice planes and exponents (one allocation)
  void* slice_dev = nullptr;
  size_t slice_bytes = 0;
  hipEvent_t ready = nullptr;     // upload finished
  hipEvent_t last_launch = nullptr;
};

struct GraphEntry {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipEvent_t done = nullptr;      // recorded after every launch of this graph
  uint64_t owner = 0;             // DescEntry::id of the descriptor set it was captured for
  uint64_t last_use = 0;
};

struct fmm_ctx {
  int device = -1;
  bool host_only = true;
  std::string last_error;
  hipStream_t internal = nullptr;
  int* d_stencil = nullptr;
  double* d_D = nullptr;                      // [892][165] derivatives up to order 8
  double* d_T[kMaxP + 1] = {};                // canonical [892][C][C] per order
  MfmaTables mfma;                            // packed tables for the matrix-core kernels
  SliceTables slice;                          // int8 table slices of FMM_EXACT_SLICE
  TreeTables tree;                            // interaction-list tables of the multi-level M2L
  std::vector<std::unique_ptr<DescEntry>> descs;
  std::unordered_map<uint64_t, GraphEntry> graphs;
  uint64_t clock = 0;
  uint64_t next_id = 0;
  int m2l_kernel = 0;                         // 0 auto, 1 reference, 2 matrix core
  int use_graph = 1;
  int tile_config = -1;
  int adjoint_form = 0;     // FMM_OPT_ADJOINT_FORM
  int p2m_window = 0;       // FMM_OPT_P2M_WINDOW
  int round_split = -1;     // FMM_OPT_ROUND_SPLIT: -1 as tuned or planned, 0 whole sub-grids, 1 parts (small batches)
  int slices = 7;           // FMM_OPT_SLICES
  // fmm_m2l_noalloc: this device's address of the static array, a pinned host
  // copy of it, and the event after its upload
  unsigned char* noalloc_dev = nullptr;
  unsigned char* noalloc_host = nullptr;
  hipEvent_t noalloc_uploaded = nullptr;
};

namespace {

fmm_status set_err(fmm_ctx* ctx, fmm_status st, const std::string& msg) {
  if (ctx) ctx->last_error = msg;
  else g_create_error = msg;
  return st;
}

fmm_status hip_err(fmm_ctx* ctx, hipError_t e, const char* what) {
  std::string msg = std::string(what) + ": " + hipGetErrorName(e) + " (" + hipGetErrorString(e) + ")";
  return set_err(ctx, e == hipErrorOutOfMemory ? FMM_ENOMEM : FMM_EHIP, msg);
}

#define HIP_TRY(ctx, call)                                   \
  do {                                                       \
    hipError_t e_ = (call);                                  \
    if (e_ != hipSuccess) return hip_err((ctx), e_, #call);  \
  } while (0)

bool aligned8(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 7u) == 0; }

fmm_status check_ctx(fmm_ctx* ctx) {
  if (!ctx) return set_err(nullptr, FMM_EINVAL, "context is NULL");
  return FMM_OK;
}

fmm_status check_desc(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub) {
  if (nsub < 0) return set_err(ctx, FMM_EINVAL, "nsub < 0");
  if (nsub > 0x7fffffff) return set_err(ctx, FMM_EINVAL, "nsub exceeds 2^31 - 1");
  if (nsub > 0 && !desc) return set_err(ctx, FMM_EINVAL, "desc is NULL");
  for (int64_t b = 0; b < nsub; ++b) {
    const fmm_subgrid& d = desc[b];
    char buf[160];
    if (d.p < 2 || d.p > kMaxP) {
      snprintf(buf, sizeof buf, "desc[%lld].p = %d not in {2,3,4}", (long long)b, d.p);
      return set_err(ctx, FMM_EINVAL, buf);
    }
    if (d.log2_inv_h < 0 || d.log2_inv_h > 2) {
      snprintf(buf, sizeof buf, "desc[%lld].log2_inv_h = %d not in [0,2]", (long long)b, d.log2_inv_h);
      return set_err(ctx, FMM_EINVAL, buf);
    }
    if (d.mask > kFullMask || !((d.mask >> kCentreBit) & 1u)) {
      snprintf(buf, sizeof buf, "desc[%lld].mask = 0x%x: needs bit 13 and no bit above 26", (long long)b, d.mask);
      return set_err(ctx, FMM_EINVAL, buf);
    }
    if (d.reserved != 0) {
      snprintf(buf, sizeof buf, "desc[%lld].reserved must be 0", (long long)b);
      return set_err(ctx, FMM_EINVAL, buf);
    }
    if (d.m_off < 0 || d.l_off < 0 || d.part_off < 0) {
      snprintf(buf, sizeof buf, "desc[%lld] has a negative offset", (long long)b);
      return set_err(ctx, FMM_EINVAL, buf);
    }
  }
  return FMM_OK;
}

fmm_status check_ptr(fmm_ctx* ctx, const void* p, const char* name, int64_t nsub) {
  if (nsub == 0) return FMM_OK;
  if (!p) return set_err(ctx, FMM_EINVAL, std::string(name) + " is NULL");
  if (!aligned8(p)) return set_err(ctx, FMM_EINVAL, std::string(name) + " is not 8-byte aligned");
  return FMM_OK;
}

fmm_status check_ppc(fmm_ctx* ctx, int32_t ppc) {
  if (ppc < 1 || ppc > 64) return set_err(ctx, FMM_EINVAL, "ppc not in [1, 64]");
  return FMM_OK;
}

fmm_status check_precision(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, fmm_precision prec) {
  if (prec != FMM_FP64 && prec != FMM_SPLIT_FP32 && prec != FMM_FP64_HARMONIC && prec != FMM_EXACT_SLICE)
    return set_err(ctx, FMM_EINVAL, "unknown precision");
  if (prec == FMM_EXACT_SLICE)
    for (int64_t b = 0; b < nsub; ++b)
      if (desc[b].p > 3) {
        char buf[120];
        snprintf(buf, sizeof buf, "FMM_EXACT_SLICE runs orders 2 and 3; desc[%lld].p = %d", (long long)b, desc[b].p);
        return set_err(ctx, FMM_EUNSUPPORTED, buf);
      }
  return FMM_OK;
}

#define CHECK_OK(expr)                    \
  do {                                    \
    fmm_status s_ = (expr);               \
    if (s_ != FMM_OK) return s_;          \
  } while (0)

// Set the context's device for the duration of a call, restore on exit.
struct DeviceGuard {
  int prev = -1;
  bool changed = false;
  hipError_t err = hipSuccess;
  explicit DeviceGuard(int dev) {
    err = hipGetDevice(&prev);
    if (err == hipSuccess && prev != dev) {
      err = hipSetDevice(dev);
      changed = err == hipSuccess;
    }
  }
  ~DeviceGuard() {
    if (changed) (void)hipSetDevice(prev);
  }
};

void free_entry(DescEntry* e) {
  if (e->last_launch) (void)hipEventSynchronize(e->last_launch);
  if (e->ready) (void)hipEventSynchronize(e->ready);
  if (e->dev) (void)hipFree(e->dev);
  if (e->pinned) (void)hipHostFree(e->pinned);
  for (CallLists& l : e->lists) {
    if (l.dev) (void)hipFree(l.dev);
    if (l.pinned) (void)hipHostFree(l.pinned);
  }
  if (e->slice_dev) (void)hipFree(e->slice_dev);
  if (e->ready) (void)hipEventDestroy(e->ready);
  if (e->last_launch) (void)hipEventDestroy(e->last_launch);
}

// Wait for the graph's last launch (on whatever stream it ran), then release it.
void destroy_graph(GraphEntry& g) {
  if (g.done) (void)hipEventSynchronize(g.done);
  if (g.exec) (void)hipGraphExecDestroy(g.exec);
  if (g.graph) (void)hipGraphDestroy(g.graph);
  if (g.done) (void)hipEventDestroy(g.done);
  g = GraphEntry{};
}

constexpr size_t kMaxDescEntries = 8;
constexpr size_t kMaxGraphs = 16;

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Sizes of a set's allocations: sets that replace each other mostly have the same
// (a new size costs hipHostMalloc 100 to 150 us, one just freed 15).
size_t alloc_size(size_t x) {
  constexpr size_t kStep = 1 << 20;
  if (x > kStep) return align_up(x, kStep);
  size_t n = 64 << 10;
  while (n < x) n *= 2;
  return n;
}

struct ListItems {
  std::vector<WorkItem> whole, cut;
  size_t off_cut() const { return align_up(sizeof(WorkItem) * whole.size(), 256); }
  size_t off_counter() const { return align_up(off_cut() + sizeof(WorkItem) * cut.size(), 256); }
  size_t bytes() const { return off_counter() + 256; }
};
// at most, for nsub sub-grids
size_t list_room(int64_t nsub, int need) {
  const int64_t cut = need >= need_adjoint(false) ? nsub * kMaxRounds
                                                  : std::min(nsub * kLevelParts[kMaxPartLevel], max_parts(nsub));
  return align_up(sizeof(WorkItem) * (size_t)nsub, 256) + align_up(sizeof(WorkItem) * (size_t)cut, 256) + 256;
}

// The items of the lists of one need, longest sub-grid first, and the plan they follow.
ListItems build_lists(const fmm_ctx* ctx, DescEntry* e, int need) {
  const bool adjoint = need >= need_adjoint(false), harmonic = need == need_forward(true) || need == need_adjoint(true);
  const int64_t nsub = (int64_t)e->host.size();
  const int num_cu = ctx->mfma.num_cu;
  ListItems li;
  li.whole.resize((size_t)nsub);
  sort_by_cost(e->host.data(), nsub, harmonic, adjoint, li.whole.data());
  if (!adjoint) {
    const StreamPlan plan = plan_stream(li.whole.data(), nsub, num_cu);
    e->plan[harmonic] = plan;
    if (plan.parts || nsub <= kMaxSplitSubgrids) {
      li.cut = li.whole;
      li.cut.resize((size_t)max_parts(nsub));
      li.cut.resize((size_t)split_items(e->host.data(), li.cut.data(), nsub, num_cu));
    }
  } else {
    const AdjointPlan plan = plan_adjoint(li.whole.data(), nsub, num_cu, harmonic);
    e->adjoint_plan[harmonic] = plan;
    if (plan.rounds)
      for (const WorkItem& it : li.whole) {
        uint32_t sets[kMaxRounds];
        const int n = adjoint_round_sets(e->host[(size_t)it.sub].p, harmonic, sets);
        for (int k = 0; k < n; ++k) li.cut.push_back(WorkItem{it.sub, (int32_t)sets[k]});
      }
  }
  whole_items(li.whole.data(), nsub);
  return li;
}

// Writes the lists at hp (host) for their copy to dp (device).
void place_lists(const ListItems& li, CallLists* l, char* hp, char* dp) {
  std::memcpy(hp, li.whole.data(), sizeof(WorkItem) * li.whole.size());
  std::memcpy(hp + li.off_cut(), li.cut.data(), sizeof(WorkItem) * li.cut.size());
  std::memset(hp + li.off_counter(), 0, 256);
  l->made = true;
  l->whole.items = reinterpret_cast<const WorkItem*>(dp);
  l->whole.count = (int)li.whole.size();
  l->whole.counter = reinterpret_cast<unsigned*>(dp + li.off_counter());
  l->cut = l->whole;
  l->cut.items = reinterpret_cast<const WorkItem*>(dp + li.off_cut());
  l->cut.count = (int)li.cut.size();
  l->cut.parts = true;
}

// Find or upload the descriptor set; builds the id lists, and for a new set the
// work lists of the call's need.
fmm_status get_desc(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, hipStream_t stream,
                    int need, DescEntry** out) {
  const size_t nbytes = sizeof(fmm_subgrid) * (size_t)nsub;
  const uint64_t h = fnv1a(desc, nbytes, fnv1a(&nsub, sizeof nsub));
  for (auto& e : ctx->descs) {
    if (e->hash == h && e->host.size() == (size_t)nsub &&
        std::memcmp(e->host.data(), desc, nbytes) == 0) {
      e->last_use = ++ctx->clock;
      // order after the previous call on this set, whatever its stream: calls
      // share the set's work-list counters (the event
      // was first recorded after the upload, so this also covers the upload)
      HIP_TRY(ctx, hipStreamWaitEvent(stream, e->last_launch, 0));
      *out = e.get();
      return FMM_OK;
    }
  }
  if (ctx->descs.size() >= kMaxDescEntries) {
    auto it = std::min_element(ctx->descs.begin(), ctx->descs.end(),
                               [](const auto& a, const auto& b) { return a->last_use < b->last_use; });
    // the graphs captured for this set refer to its work list: drop those (each
    // waits for its own last launch); the other sets' graphs stay
    const uint64_t owner = (*it)->id;
    for (auto g = ctx->graphs.begin(); g != ctx->graphs.end();) {
      if (g->second.owner == owner) {
        destroy_graph(g->second);
        g = ctx->graphs.erase(g);
      } else {
        ++g;
      }
    }
    free_entry(it->get());
    ctx->descs.erase(it);
  }
  auto e = std::make_unique<DescEntry>();
  e->host.assign(desc, desc + nsub);
  e->hash = h;
  e->id = ++ctx->next_id;
  e->last_use = ++ctx->clock;
  // layout: descriptors | ids per order | the call's work lists | room for the others
  std::vector<int> ids[kMaxP + 1];
  for (int64_t b = 0; b < nsub; ++b) {
    ids[desc[b].p].push_back((int)b);
    if (desc[b].part_off & 1) e->part_even = false;
  }
  size_t off_desc = 0;
  size_t off = align_up(nbytes, 256);
  size_t off_ids[kMaxP + 1] = {};
  for (int p = 2; p <= kMaxP; ++p) {
    off_ids[p] = off;
    off = align_up(off + sizeof(int) * ids[p].size(), 256);
  }
  ListItems lists;
  if (need != kNeedNone) {
    lists = build_lists(ctx, e.get(), need);
    e->room[need] = off;
    off = align_up(off + lists.bytes(), 256);
  }
  const size_t upload = off;
  for (int k = 0; k < 4 && nsub <= kRoomSubgrids; ++k)
    if (k != need) {
      e->room[k] = off;
      off += list_room(nsub, k);
    }
  e->bytes = alloc_size(off);
  HIP_TRY(ctx, hipMalloc(&e->dev, e->bytes));
  HIP_TRY(ctx, hipHostMalloc(&e->pinned, e->bytes, hipHostMallocDefault));
  char* hp = static_cast<char*>(e->pinned);
  std::memcpy(hp + off_desc, desc, nbytes);
  for (int p = 2; p <= kMaxP; ++p) std::memcpy(hp + off_ids[p], ids[p].data(), sizeof(int) * ids[p].size());
  char* dp = static_cast<char*>(e->dev);
  e->d_desc = reinterpret_cast<DevDesc*>(dp + off_desc);
  for (int p = 2; p <= kMaxP; ++p) {
    e->d_ids[p] = reinterpret_cast<int*>(dp + off_ids[p]);
    e->count[p] = (int)ids[p].size();
  }
  if (need != kNeedNone) place_lists(lists, &e->lists[need], hp + e->room[need], dp + e->room[need]);
  HIP_TRY(ctx, hipEventCreateWithFlags(&e->ready, hipEventDisableTiming));
  HIP_TRY(ctx, hipEventCreateWithFlags(&e->last_launch, hipEventDisableTiming));
  HIP_TRY(ctx, hipMemcpyAsync(e->dev, e->pinned, upload, hipMemcpyHostToDevice, stream));
  HIP_TRY(ctx, hipEventRecord(e->ready, stream));
  HIP_TRY(ctx, hipEventRecord(e->last_launch, stream));
  *out = e.get();
  ctx->descs.push_back(std::move(e));
  return FMM_OK;
}

// Makes the lists of a need that the set's first call did not have, copied on the
// caller's stream. A caller whose stream is being captured gets them at once (the
// captured work runs later, and other calls may use them before).
fmm_status ensure_lists(fmm_ctx* ctx, DescEntry* e, int need, hipStream_t stream) {
  CallLists* l = &e->lists[need];
  if (l->made) return FMM_OK;
  const ListItems li = build_lists(ctx, e, need);
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (stream) HIP_TRY(ctx, hipStreamIsCapturing(stream, &status));
  const bool capturing = status == hipStreamCaptureStatusActive;
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;   // lets this thread allocate and wait while it captures
  if (capturing) HIP_TRY(ctx, hipThreadExchangeStreamCaptureMode(&mode));
  hipError_t err = hipSuccess;
  char *hp = static_cast<char*>(e->pinned) + e->room[need], *dp = static_cast<char*>(e->dev) + e->room[need];
  if (!e->room[need]) {
    err = hipMalloc(&l->dev, alloc_size(li.bytes()));
    if (err == hipSuccess) err = hipHostMalloc(&l->pinned, alloc_size(li.bytes()), hipHostMallocDefault);
    hp = static_cast<char*>(l->pinned);
    dp = static_cast<char*>(l->dev);
  }
  if (err == hipSuccess) {
    place_lists(li, l, hp, dp);
    err = hipMemcpyAsync(dp, hp, li.bytes(), hipMemcpyHostToDevice, capturing ? ctx->internal : stream);
  }
  if (err == hipSuccess)
    err = capturing ? hipStreamSynchronize(ctx->internal) : hipEventRecord(e->last_launch, stream);
  if (capturing) (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (err != hipSuccess) {
    if (l->dev) (void)hipFree(l->dev);
    if (l->pinned) (void)hipHostFree(l->pinned);
    *l = CallLists{};
    return hip_err(ctx, err, "work lists");
  }
  return FMM_OK;
}

fmm_status mark_used(fmm_ctx* ctx, DescEntry* e, hipStream_t stream) {
  HIP_TRY(ctx, hipEventRecord(e->last_launch, stream));
  return FMM_OK;
}

}  // namespace

extern "C" {

const char* fmm_status_string(fmm_status s) {
  if (s <= 0 && s >= -4) return kStatusStrings[-s];
  return "unknown fmm_status";
}

const char* fmm_last_error(const fmm_ctx* ctx) {
  return ctx ? ctx->last_error.c_str() : g_create_error.c_str();
}

fmm_status fmm_stencil(int32_t* count, int32_t* offsets) {
  if (!count) return set_err(nullptr, FMM_EINVAL, "count is NULL");
  const auto& s = stencil_host();
  *count = (int32_t)(s.size() / 3);
  if (offsets) std::memcpy(offsets, s.data(), s.size() * sizeof(int32_t));
  return FMM_OK;
}

fmm_status fmm_pair_count(const fmm_subgrid* desc, int64_t nsub, int64_t* pairs) {
  if (!pairs) return set_err(nullptr, FMM_EINVAL, "pairs is NULL");
  CHECK_OK(check_desc(nullptr, desc, nsub));
  int64_t n = 0;
  for (int64_t b = 0; b < nsub; ++b) n += pairs_of_mask(desc[b].mask);
  *pairs = n;
  return FMM_OK;
}

fmm_status fmm_create(fmm_ctx** out, int32_t device) {
  if (!out) return set_err(nullptr, FMM_EINVAL, "out is NULL");
  *out = nullptr;
  if (device < -1) return set_err(nullptr, FMM_EINVAL, "device < -1");
  auto ctx = std::make_unique<fmm_ctx>();
  if (device == -1) {
    *out = ctx.release();
    return FMM_OK;
  }
  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess) return hip_err(nullptr, e, "hipGetDeviceCount");
  if (device >= ndev) return set_err(nullptr, FMM_EINVAL, "device index out of range");
  ctx->device = device;
  ctx->host_only = false;
  DeviceGuard guard(device);
  if (guard.err != hipSuccess) return hip_err(nullptr, guard.err, "hipSetDevice");
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, device);
  if (e != hipSuccess) return hip_err(nullptr, e, "hipGetDeviceProperties");
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return set_err(nullptr, FMM_EUNSUPPORTED, std::string("device is ") + prop.gcnArchName + ", library is built for gfx950");
  fmm_ctx* c = ctx.get();
  auto fail = [&](hipError_t err, const char* what) {
    fmm_status st = hip_err(c, err, what);
    g_create_error = c->last_error;
    fmm_destroy(ctx.release());
    return st;
  };
#define CREATE_TRY(call) do { hipError_t e_ = (call); if (e_ != hipSuccess) return fail(e_, #call); } while (0)
  CREATE_TRY(hipStreamCreateWithFlags(&c->internal, hipStreamNonBlocking));
  const auto& st = stencil_host();
  CREATE_TRY(hipMalloc(&c->d_stencil, st.size() * sizeof(int)));
  CREATE_TRY(hipMemcpyAsync(c->d_stencil, st.data(), st.size() * sizeof(int), hipMemcpyHostToDevice, c->internal));
  CREATE_TRY(hipMalloc(&c->d_D, sizeof(double) * kNStencil * ncomp(kMaxOrderD)));
  const std::vector<double> hD = host_derivative_tables(st.data(), kNStencil, kMaxOrderD);
  CREATE_TRY(hipMemcpyAsync(c->d_D, hD.data(), sizeof(double) * hD.size(), hipMemcpyHostToDevice, c->internal));
  for (int p = 2; p <= kMaxP; ++p) {
    const int C = ncomp(p);
    CREATE_TRY(hipMalloc(&c->d_T[p], sizeof(double) * kNStencil * C * C));
    CREATE_TRY(launch_build_tensors(c->d_D, kMaxOrderD, p, c->d_T[p], c->internal));
  }
  CREATE_TRY(mfma_tables_create(&c->mfma, c->d_T, c->d_stencil, c->internal));
  CREATE_TRY(slice_tables_create(&c->slice, c->d_T, c->internal));
  CREATE_TRY(tree_tables_create(&c->tree, c->d_T, st.data(), (int)(st.size() / 3), c->internal));
  // fmm_m2l_noalloc: the device's address of the static array (the device is current)
  CREATE_TRY(hipGetSymbolAddress(reinterpret_cast<void**>(&c->noalloc_dev), HIP_SYMBOL(scratch)));
  CREATE_TRY(hipHostMalloc(reinterpret_cast<void**>(&c->noalloc_host), kNoAllocBytes, hipHostMallocDefault));
  CREATE_TRY(hipEventCreateWithFlags(&c->noalloc_uploaded, hipEventDisableTiming));
  (void)pairs_of_mask(0);   // the work-list builder's table is made here, not in a compute call
  CREATE_TRY(hipStreamSynchronize(c->internal));
#undef CREATE_TRY
  *out = ctx.release();
  return FMM_OK;
}

fmm_status fmm_destroy(fmm_ctx* ctx) {
  if (!ctx) return FMM_OK;
  if (!ctx->host_only) {
    DeviceGuard guard(ctx->device);
    (void)hipDeviceSynchronize();
    for (auto& g : ctx->graphs) destroy_graph(g.second);
    for (auto& e : ctx->descs) free_entry(e.get());
    mfma_tables_destroy(&ctx->mfma);
    slice_tables_destroy(&ctx->slice);
    tree_tables_destroy(&ctx->tree);
    for (int p = 0; p <= kMaxP; ++p)
      if (ctx->d_T[p]) (void)hipFree(ctx->d_T[p]);
    if (ctx->d_D) (void)hipFree(ctx->d_D);
    if (ctx->d_stencil) (void)hipFree(ctx->d_stencil);
    if (ctx->noalloc_host) (void)hipHostFree(ctx->noalloc_host);
    if (ctx->noalloc_uploaded) (void)hipEventDestroy(ctx->noalloc_uploaded);
    if (ctx->internal) (void)hipStreamDestroy(ctx->internal);
  }
  delete ctx;
  return FMM_OK;
}

fmm_status fmm_set_option(fmm_ctx* ctx, int32_t option, int64_t value) {
  CHECK_OK(check_ctx(ctx));
  switch (option) {
    case FMM_OPT_M2L_KERNEL:
      if (value < 0 || value > 2) return set_err(ctx, FMM_EINVAL, "FMM_OPT_M2L_KERNEL value not in [0,2]");
      ctx->m2l_kernel = (int)value;
      return FMM_OK;
    case FMM_OPT_USE_GRAPH:
      if (value != 0 && value != 1) return set_err(ctx, FMM_EINVAL, "FMM_OPT_USE_GRAPH value not 0/1");
      ctx->use_graph = (int)value;
      return FMM_OK;
    case FMM_OPT_P2M_WINDOW:
      if (value != 0 && value != 1) return set_err(ctx, FMM_EINVAL, "FMM_OPT_P2M_WINDOW value not 0/1");
      ctx->p2m_window = (int)value;
      return FMM_OK;
    case FMM_OPT_ROUND_SPLIT:
      if (value < -1 || value > 1) return set_err(ctx, FMM_EINVAL, "FMM_OPT_ROUND_SPLIT value not -1/0/1");
      ctx->round_split = (int)value;
      return FMM_OK;
    case FMM_OPT_SLICES:
      if (value < kSliceMin || value > kSliceMax) return set_err(ctx, FMM_EINVAL, "FMM_OPT_SLICES value not in [6,8]");
      ctx->slices = (int)value;
      return FMM_OK;
    case FMM_OPT_ADJOINT_FORM:
      if (value != 0 && value != 1) return set_err(ctx, FMM_EINVAL, "FMM_OPT_ADJOINT_FORM value not 0/1");
      ctx->adjoint_form = (int)value;
      return FMM_OK;
    case FMM_OPT_TILE_CONFIG:
      if (value < -1 || value >= mfma_num_configs()) return set_err(ctx, FMM_EINVAL, "FMM_OPT_TILE_CONFIG out of range");
      ctx->tile_config = (int)value;
      return FMM_OK;
    default:
      return set_err(ctx, FMM_EINVAL, "unknown option");
  }
}

fmm_status fmm_p2m(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* pos,
                   const double* mass, int32_t ppc, double* M, void* stream) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ppc(ctx, ppc));
  CHECK_OK(check_ptr(ctx, pos, "pos", nsub));
  CHECK_OK(check_ptr(ctx, mass, "mass", nsub));
  CHECK_OK(check_ptr(ctx, M, "M", nsub));
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) return FMM_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  DescEntry* e = nullptr;
  CHECK_OK(get_desc(ctx, desc, nsub, s, kNeedNone, &e));
  HIP_TRY(ctx, launch_p2m(e->d_desc, nsub, e->d_ids, e->count, pos, mass, ppc, M, e->part_even,
                          ctx->p2m_window != 0, s));
  return mark_used(ctx, e, s);
}

fmm_status fmm_p2m_backward(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* pos,
                            int32_t ppc, const double* dM, double* dmass, void* stream) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ppc(ctx, ppc));
  CHECK_OK(check_ptr(ctx, pos, "pos", nsub));
  CHECK_OK(check_ptr(ctx, dM, "dM", nsub));
  CHECK_OK(check_ptr(ctx, dmass, "dmass", nsub));
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) return FMM_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  DescEntry* e = nullptr;
  CHECK_OK(get_desc(ctx, desc, nsub, s, kNeedNone, &e));
  HIP_TRY(ctx, launch_p2m_backward(e->d_desc, nsub, e->d_ids, e->count, pos, ppc, dM, dmass, e->part_even, s));
  return mark_used(ctx, e, s);
}

fmm_status fmm_evaluate(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* pos,
                        const double* mass, int32_t ppc, const double* L, double* out,
                        void* stream) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ppc(ctx, ppc));
  CHECK_OK(check_ptr(ctx, pos, "pos", nsub));
  CHECK_OK(check_ptr(ctx, mass, "mass", nsub));
  CHECK_OK(check_ptr(ctx, L, "L", nsub));
  CHECK_OK(check_ptr(ctx, out, "out", nsub));
  // one workgroup of 256 threads per target z-plane: the grid's thread count fits 32 bits
  if (nsub > (int64_t)1 << 21) return set_err(ctx, FMM_EINVAL, "nsub exceeds 2^21 for fmm_evaluate");
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) return FMM_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  DescEntry* e = nullptr;
  CHECK_OK(get_desc(ctx, desc, nsub, s, kNeedNone, &e));
  HIP_TRY(ctx, launch_evaluate(e->d_desc, nsub, pos, mass, ppc, L, out, s));
  return mark_used(ctx, e, s);
}

// ---------------------------------------------------------------------------
// multi-level iteration on a uniform octree

static fmm_status check_tree(fmm_ctx* ctx, const fmm_tree* t) {
  if (!t) return set_err(ctx, FMM_EINVAL, "tree is NULL");
  if (t->p < 2 || t->p > kMaxP) return set_err(ctx, FMM_EINVAL, "tree.p not in {2,3,4}");
  if (t->n < 8 || t->n > 128 || (t->n & (t->n - 1)))
    return set_err(ctx, FMM_EINVAL, "tree.n must be 8, 16, 32, 64 or 128");
  if (t->ppc < 1 || t->ppc > 64) return set_err(ctx, FMM_EINVAL, "tree.ppc not in [1, 64]");
  if (t->log2_h < -4 || t->log2_h > 4) return set_err(ctx, FMM_EINVAL, "tree.log2_h not in [-4, 4]");
  if (t->harmonic != 0 && t->harmonic != 1) return set_err(ctx, FMM_EINVAL, "tree.harmonic not 0/1");
  return FMM_OK;
}

static int tree_nlevels(int n) {
  int l = 1;
  for (int m = n; m > 4; m /= 2) ++l;
  return l;
}

// element offset of level l in a workspace
static int64_t tree_level_off(const fmm_tree* t, int l) {
  const int64_t C = ncomp(t->p);
  int64_t off = 0;
  for (int i = 0, m = t->n; i < l; ++i, m /= 2) off += C * m * m * m;
  return off;
}

static fmm_status tree_begin(fmm_ctx* ctx, const fmm_tree* t) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_tree(ctx, t));
  return FMM_OK;
}

static fmm_status tree_device(fmm_ctx* ctx) {
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  return FMM_OK;
}

fmm_status fmm_tree_size(const fmm_tree* tree, int32_t* levels, int64_t* elems) {
  CHECK_OK(check_tree(nullptr, tree));
  const int nl = tree_nlevels(tree->n);
  if (levels) *levels = nl;
  if (elems) *elems = tree_level_off(tree, nl);
  return FMM_OK;
}

static fmm_status tree_upward(fmm_ctx* ctx, const fmm_tree* t, const double* pos, const double* mass,
                              double* M, hipStream_t s) {
  HIP_TRY(ctx, launch_tree_p2m(t->p, pos, mass, t->ppc, t->n, ldexp(1.0, t->log2_h), M, s));
  const int nl = tree_nlevels(t->n);
  for (int l = 0, m = t->n; l + 1 < nl; ++l, m /= 2)
    HIP_TRY(ctx, launch_tree_m2m(t->p, M + tree_level_off(t, l), M + tree_level_off(t, l + 1), m,
                                 ldexp(1.0, t->log2_h + l), s));
  return FMM_OK;
}

static fmm_status tree_m2l(fmm_ctx* ctx, const fmm_tree* t, const double* M, double* L, hipStream_t s) {
  const int nl = tree_nlevels(t->n);
  int n[8], lg[8];
  int64_t off[8];
  for (int l = 0, m = t->n; l < nl; ++l, m /= 2) {
    n[l] = m;
    lg[l] = t->log2_h + l;
    off[l] = tree_level_off(t, l);
  }
  HIP_TRY(ctx, launch_tree_m2l(t->p, ctx->tree, ctx->mfma, t->harmonic != 0, M, L, nl, n, lg, off, s));
  return FMM_OK;
}

static fmm_status tree_downward(fmm_ctx* ctx, const fmm_tree* t, double* L, hipStream_t s) {
  const int nl = tree_nlevels(t->n);
  for (int l = nl - 2; l >= 0; --l)
    HIP_TRY(ctx, launch_tree_l2l(t->p, L + tree_level_off(t, l + 1), L + tree_level_off(t, l),
                                 t->n >> l, ldexp(1.0, t->log2_h + l), s));
  return FMM_OK;
}

fmm_status fmm_tree_upward(fmm_ctx* ctx, const fmm_tree* tree, const double* pos, const double* mass,
                           double* M, void* stream) {
  CHECK_OK(tree_begin(ctx, tree));
  CHECK_OK(check_ptr(ctx, pos, "pos", 1));
  CHECK_OK(check_ptr(ctx, mass, "mass", 1));
  CHECK_OK(check_ptr(ctx, M, "M", 1));
  CHECK_OK(tree_device(ctx));
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  return tree_upward(ctx, tree, pos, mass, M, static_cast<hipStream_t>(stream));
}

fmm_status fmm_tree_m2l(fmm_ctx* ctx, const fmm_tree* tree, const double* M, double* L, void* stream) {
  CHECK_OK(tree_begin(ctx, tree));
  CHECK_OK(check_ptr(ctx, M, "M", 1));
  CHECK_OK(check_ptr(ctx, L, "L", 1));
  CHECK_OK(tree_device(ctx));
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  return tree_m2l(ctx, tree, M, L, static_cast<hipStream_t>(stream));
}

fmm_status fmm_tree_downward(fmm_ctx* ctx, const fmm_tree* tree, double* L, void* stream) {
  CHECK_OK(tree_begin(ctx, tree));
  CHECK_OK(check_ptr(ctx, L, "L", 1));
  CHECK_OK(tree_device(ctx));
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  return tree_downward(ctx, tree, L, static_cast<hipStream_t>(stream));
}

fmm_status fmm_tree_evaluate(fmm_ctx* ctx, const fmm_tree* tree, const double* pos, const double* mass,
                             const double* L, double* out, void* stream) {
  CHECK_OK(tree_begin(ctx, tree));
  CHECK_OK(check_ptr(ctx, pos, "pos", 1));
  CHECK_OK(check_ptr(ctx, mass, "mass", 1));
  CHECK_OK(check_ptr(ctx, L, "L", 1));
  CHECK_OK(check_ptr(ctx, out, "out", 1));
  CHECK_OK(tree_device(ctx));
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  HIP_TRY(ctx, launch_evaluate_grid(tree->p, tree->n, ldexp(1.0, tree->log2_h), pos, mass, tree->ppc, L,
                                    out, static_cast<hipStream_t>(stream)));
  return FMM_OK;
}

fmm_status fmm_tree_solve(fmm_ctx* ctx, const fmm_tree* tree, const double* pos, const double* mass,
                          double* M, double* L, double* out, void* stream) {
  CHECK_OK(tree_begin(ctx, tree));
  CHECK_OK(check_ptr(ctx, pos, "pos", 1));
  CHECK_OK(check_ptr(ctx, mass, "mass", 1));
  CHECK_OK(check_ptr(ctx, M, "M", 1));
  CHECK_OK(check_ptr(ctx, L, "L", 1));
  CHECK_OK(check_ptr(ctx, out, "out", 1));
  CHECK_OK(tree_device(ctx));
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  hipStream_t s = static_cast<hipStream_t>(stream);
  CHECK_OK(tree_upward(ctx, tree, pos, mass, M, s));
  CHECK_OK(tree_m2l(ctx, tree, M, L, s));
  CHECK_OK(tree_downward(ctx, tree, L, s));
  HIP_TRY(ctx, launch_evaluate_grid(tree->p, tree->n, ldexp(1.0, tree->log2_h), pos, mass, tree->ppc, L,
                                    out, s));
  return FMM_OK;
}

static fmm_status run_ref(fmm_ctx* ctx, DescEntry* e, bool backward, const double* src, double* out,
                          hipStream_t s) {
  for (int p = 2; p <= kMaxP; ++p)
    HIP_TRY(ctx, launch_m2l_ref(p, backward, e->d_desc, e->d_ids[p], e->count[p], ctx->d_stencil,
                                ctx->d_T[p], src, out, s));
  return FMM_OK;
}

// Launch a persistent matrix-core kernel over whole sub-grids, through a cached
// graph if enabled.
static fmm_status run_mfma(fmm_ctx* ctx, DescEntry* e, const double* M, double* L,
                           fmm_precision prec, int cfg, hipStream_t s) {
  WorkList wl = e->lists[need_forward(false)].whole;
  wl.counter += 1;
  if (!ctx->use_graph) {
    HIP_TRY(ctx, launch_m2l_mfma(ctx->mfma, wl, e->d_desc, M, L, prec, cfg, s));
    return FMM_OK;
  }
  uint64_t key = fnv1a(&e->id, sizeof e->id);
  key = fnv1a(&M, sizeof M, key);
  key = fnv1a(&L, sizeof L, key);
  key = fnv1a(&prec, sizeof prec, key);
  key = fnv1a(&cfg, sizeof cfg, key);
  auto it = ctx->graphs.find(key);
  if (it == ctx->graphs.end()) {
    if (ctx->graphs.size() >= kMaxGraphs) {
      // the least recently used graph; its own last launch (on any stream) is
      // waited for before it is released
      auto victim = std::min_element(ctx->graphs.begin(), ctx->graphs.end(),
                                     [](const auto& a, const auto& b) { return a.second.last_use < b.second.last_use; });
      destroy_graph(victim->second);
      ctx->graphs.erase(victim);
    }
    GraphEntry g;
    g.owner = e->id;
    HIP_TRY(ctx, hipStreamBeginCapture(ctx->internal, hipStreamCaptureModeThreadLocal));
    hipError_t le = launch_m2l_mfma(ctx->mfma, wl, e->d_desc, M, L, prec, cfg, ctx->internal);
    hipError_t ce = hipStreamEndCapture(ctx->internal, &g.graph);
    if (le != hipSuccess || ce != hipSuccess) {
      if (g.graph) (void)hipGraphDestroy(g.graph);
      return le != hipSuccess ? hip_err(ctx, le, "launch_m2l_mfma (capture)")
                              : hip_err(ctx, ce, "hipStreamEndCapture");
    }
    hipError_t ie = hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0);
    if (ie == hipSuccess) ie = hipEventCreateWithFlags(&g.done, hipEventDisableTiming);
    if (ie != hipSuccess) {
      destroy_graph(g);
      return hip_err(ctx, ie, "hipGraphInstantiate");
    }
    it = ctx->graphs.emplace(key, g).first;
  }
  it->second.last_use = ++ctx->clock;
  HIP_TRY(ctx, hipGraphLaunch(it->second.exec, s));
  HIP_TRY(ctx, hipEventRecord(it->second.done, s));
  return FMM_OK;
}

// FMM_EXACT_SLICE: the slice planes and exponents of the set (allocated on first
// use, and again if more slices are asked for), then the two kernels
static fmm_status run_slice(fmm_ctx* ctx, DescEntry* e, const double* M, double* L, hipStream_t s) {
  CHECK_OK(ensure_lists(ctx, e, need_forward(true), s));
  const int64_t nsub = (int64_t)e->host.size();
  const size_t planes = align_up((size_t)nsub * ctx->slices * kSlicePlane, 256);
  const size_t bytes = planes + sizeof(int32_t) * (size_t)nsub;
  if (e->slice_bytes < bytes) {
    if (e->slice_dev) {
      // the previous launches on this set read the old buffer
      HIP_TRY(ctx, hipEventSynchronize(e->last_launch));
      (void)hipFree(e->slice_dev);
      e->slice_dev = nullptr;
      e->slice_bytes = 0;
    }
    HIP_TRY(ctx, hipMalloc(&e->slice_dev, bytes));
    e->slice_bytes = bytes;
  }
  int8_t* pl = static_cast<int8_t*>(e->slice_dev);
  int32_t* ex = reinterpret_cast<int32_t*>(pl + planes);
  HIP_TRY(ctx, launch_m2l_slice(ctx->mfma, ctx->slice, e->lists[need_forward(true)].whole, e->d_desc, nsub, M, L, ctx->slices, pl, ex, s));
  return FMM_OK;
}

// FMM_OPT_ROUND_SPLIT: whole sub-grids, parts of them (small batches), or as the
// autotuner found (tuned) or the plan expects
static bool takes_parts(const fmm_ctx* ctx, int64_t nsub, const StreamPlan& plan, int tuned) {
  if (ctx->round_split == 0) return false;
  if (ctx->round_split == 1 && nsub <= kMaxSplitSubgrids) return true;
  return tuned < 0 ? plan.parts : tuned == 1;
}

// (its forward lists made)
static const WorkList& stream_list(const fmm_ctx* ctx, const DescEntry* e, bool harmonic) {
  const CallLists& l = e->lists[need_forward(harmonic)];
  const int tuned = e->tuned_parts[harmonic ? FMM_FP64_HARMONIC : FMM_FP64];
  return takes_parts(ctx, (int64_t)e->host.size(), e->plan[harmonic], tuned) ? l.cut : l.whole;
}

// The M2L of one call: reference kernel, exact slices, the streamed forward, or
// another matrix-core kernel over whole sub-grids.
static fmm_status run_m2l(fmm_ctx* ctx, DescEntry* e, const double* M, double* L, fmm_precision prec,
                          int cfg, hipStream_t s) {
  if (ctx->m2l_kernel == 1) return run_ref(ctx, e, false, M, L, s);
  if (prec == FMM_EXACT_SLICE) return run_slice(ctx, e, M, L, s);
  const bool harm = prec == FMM_FP64_HARMONIC;
  CHECK_OK(ensure_lists(ctx, e, need_forward(harm), s));
  if (mfma_config_streams(cfg)) {
    HIP_TRY(ctx, launch_m2l_stream(ctx->mfma, stream_list(ctx, e, harm), e->d_desc, M, L, harm, s));
    return FMM_OK;
  }
  if (prec == FMM_SPLIT_FP32) {
    HIP_TRY(ctx, launch_m2l_split(ctx->mfma, e->lists[need_forward(false)].whole, e->d_desc, M, L, s));
    return FMM_OK;
  }
  return run_mfma(ctx, e, M, L, prec, cfg, s);
}

static int pick_config(const fmm_ctx* ctx, const DescEntry* e, fmm_precision prec) {
  if (ctx->tile_config >= 0) return ctx->tile_config;
  if (e && e->tuned[prec] >= 0) return e->tuned[prec];
  return mfma_default_config(prec);
}

fmm_status fmm_m2l(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* M, double* L,
                   fmm_precision prec, void* stream) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ptr(ctx, M, "M", nsub));
  CHECK_OK(check_ptr(ctx, L, "L", nsub));
  CHECK_OK(check_precision(ctx, desc, nsub, prec));
  if (prec != FMM_FP64 && ctx->m2l_kernel == 1)
    return set_err(ctx, FMM_EINVAL, "the reference kernel computes FMM_FP64 only");
  if (ctx->m2l_kernel != 1 && ctx->tile_config >= 0 && !mfma_config_supports(ctx->tile_config, prec))
    return set_err(ctx, FMM_EINVAL, "FMM_OPT_TILE_CONFIG selects a configuration of the other precision");
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) return FMM_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  DescEntry* e = nullptr;
  const int need = ctx->m2l_kernel == 1 ? kNeedNone : need_forward(prec == FMM_FP64_HARMONIC || prec == FMM_EXACT_SLICE);
  CHECK_OK(get_desc(ctx, desc, nsub, s, need, &e));
  CHECK_OK(run_m2l(ctx, e, M, L, prec, pick_config(ctx, e, prec), s));
  return mark_used(ctx, e, s);
}

fmm_status fmm_m2l_noalloc(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* M,
                           double* L, fmm_precision prec, void* stream) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ptr(ctx, M, "M", nsub));
  CHECK_OK(check_ptr(ctx, L, "L", nsub));
  CHECK_OK(check_precision(ctx, desc, nsub, prec));
  if (nsub > FMM_NOALLOC_MAX_SUBGRIDS)
    return set_err(ctx, FMM_EINVAL, "fmm_m2l_noalloc: nsub exceeds FMM_NOALLOC_MAX_SUBGRIDS (16384)");
  if (prec == FMM_EXACT_SLICE)
    return set_err(ctx, FMM_EUNSUPPORTED, "fmm_m2l_noalloc: FMM_EXACT_SLICE needs slice buffers (use fmm_m2l)");
  if (ctx->m2l_kernel == 1)
    return set_err(ctx, FMM_EUNSUPPORTED, "fmm_m2l_noalloc runs the matrix-core kernels only");
  if (ctx->tile_config >= 0 && !mfma_config_supports(ctx->tile_config, prec))
    return set_err(ctx, FMM_EINVAL, "FMM_OPT_TILE_CONFIG selects a configuration of the other precision");
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) return FMM_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  // the pinned copy is rewritten only after the previous call's upload out of it
  HIP_TRY(ctx, hipEventSynchronize(ctx->noalloc_uploaded));
  unsigned char* hp = ctx->noalloc_host;
  std::memcpy(hp, desc, sizeof(fmm_subgrid) * (size_t)nsub);
  // the upload clears the counter, whatever earlier calls left in it (every
  // context's calls on the device share it, and overlapping ones may leave any value)
  std::memset(hp + kNoAllocCounterOff, 0, kNoAllocWorkOff - kNoAllocCounterOff);
  WorkItem* items = reinterpret_cast<WorkItem*>(hp + kNoAllocWorkOff);
  const bool harm = prec == FMM_FP64_HARMONIC;
  const int cfg = pick_config(ctx, nullptr, prec);
  const bool streams = mfma_config_streams(cfg);
  int64_t count = nsub;
  WorkList wl;
  sort_by_cost(desc, nsub, harm, false, items);
  wl.parts = streams && takes_parts(ctx, nsub, plan_stream(items, nsub, ctx->mfma.num_cu), -1);
  if (wl.parts) count = split_items(desc, items, nsub, ctx->mfma.num_cu);
  else whole_items(items, nsub);
  const size_t used = kNoAllocWorkOff + sizeof(WorkItem) * (size_t)count;
  HIP_TRY(ctx, hipMemcpyAsync(ctx->noalloc_dev, hp, used, hipMemcpyHostToDevice, s));
  HIP_TRY(ctx, hipEventRecord(ctx->noalloc_uploaded, s));
  wl.items = reinterpret_cast<const WorkItem*>(ctx->noalloc_dev + kNoAllocWorkOff);
  wl.count = (int)count;
  wl.counter = reinterpret_cast<unsigned*>(ctx->noalloc_dev + kNoAllocCounterOff);
  const DevDesc* d_desc = reinterpret_cast<const DevDesc*>(ctx->noalloc_dev);
  if (streams) HIP_TRY(ctx, launch_m2l_stream(ctx->mfma, wl, d_desc, M, L, harm, s));
  else if (prec == FMM_SPLIT_FP32) HIP_TRY(ctx, launch_m2l_split(ctx->mfma, wl, d_desc, M, L, s));
  else HIP_TRY(ctx, launch_m2l_mfma(ctx->mfma, wl, d_desc, M, L, prec, cfg, s));
  return FMM_OK;
}

fmm_status fmm_p2m_m2l(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* pos,
                       const double* mass, int32_t ppc, double* M, double* L, fmm_precision prec,
                       void* stream) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ppc(ctx, ppc));
  CHECK_OK(check_ptr(ctx, pos, "pos", nsub));
  CHECK_OK(check_ptr(ctx, mass, "mass", nsub));
  CHECK_OK(check_ptr(ctx, M, "M", nsub));
  CHECK_OK(check_ptr(ctx, L, "L", nsub));
  CHECK_OK(check_precision(ctx, desc, nsub, prec));
  if (prec != FMM_FP64 && ctx->m2l_kernel == 1)
    return set_err(ctx, FMM_EINVAL, "the reference kernel computes FMM_FP64 only");
  if (ctx->m2l_kernel != 1 && ctx->tile_config >= 0 && !mfma_config_supports(ctx->tile_config, prec))
    return set_err(ctx, FMM_EINVAL, "FMM_OPT_TILE_CONFIG selects a configuration of the other precision");
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) return FMM_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  DescEntry* e = nullptr;
  const int need = ctx->m2l_kernel == 1 ? kNeedNone : need_forward(prec == FMM_FP64_HARMONIC || prec == FMM_EXACT_SLICE);
  CHECK_OK(get_desc(ctx, desc, nsub, s, need, &e));
  const int cfg = pick_config(ctx, e, prec);
  const bool aligned = ((reinterpret_cast<uintptr_t>(pos) | reinterpret_cast<uintptr_t>(mass)) & 15u) == 0;
  // (moments in the M2L's launch where the plan expects that to be faster)
  const bool harm = prec == FMM_FP64_HARMONIC;
  bool fuse = ctx->m2l_kernel != 1 && ppc == 8 && e->part_even && aligned && mfma_config_streams(cfg);
  if (fuse) {
    CHECK_OK(ensure_lists(ctx, e, need_forward(harm), s));
    fuse = e->plan[harm].fuse;
  }
  if (fuse) {
    HIP_TRY(ctx, launch_m2l_stream(ctx->mfma, e->lists[need_forward(harm)].whole, e->d_desc, M, L, harm, s, pos, mass, M));
  } else {
    HIP_TRY(ctx, launch_p2m(e->d_desc, nsub, e->d_ids, e->count, pos, mass, ppc, M, e->part_even, true, s));
    CHECK_OK(run_m2l(ctx, e, M, L, prec, cfg, s));
  }
  return mark_used(ctx, e, s);
}

// (its adjoint lists made)
static const WorkList& adjoint_list(const DescEntry* e, bool harmonic) {
  const CallLists& l = e->lists[need_adjoint(harmonic)];
  return e->adjoint_plan[harmonic].rounds ? l.cut : l.whole;
}

fmm_status fmm_m2l_backward(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* dL,
                            double* dM, void* stream) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ptr(ctx, dL, "dL", nsub));
  CHECK_OK(check_ptr(ctx, dM, "dM", nsub));
  if (ctx->adjoint_form == 1 && ctx->m2l_kernel == 1)
    return set_err(ctx, FMM_EINVAL, "the reference kernel computes the dense adjoint only");
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) return FMM_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  DescEntry* e = nullptr;
  const int need = ctx->m2l_kernel == 1 ? kNeedNone : need_adjoint(ctx->adjoint_form == 1);
  CHECK_OK(get_desc(ctx, desc, nsub, s, need, &e));
  if (ctx->m2l_kernel == 1) {
    CHECK_OK(run_ref(ctx, e, true, dL, dM, s));
  } else {
    CHECK_OK(ensure_lists(ctx, e, need_adjoint(ctx->adjoint_form == 1), s));
    HIP_TRY(ctx, launch_m2l_mfma_backward(ctx->mfma, adjoint_list(e, ctx->adjoint_form == 1), e->d_desc, dL, dM,
                                          ctx->adjoint_form == 1, s));
  }
  return mark_used(ctx, e, s);
}

fmm_status fmm_m2l_p2m_backward(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* pos,
                                int32_t ppc, const double* dL, double* dM, double* dmass, void* stream) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ppc(ctx, ppc));
  CHECK_OK(check_ptr(ctx, pos, "pos", nsub));
  CHECK_OK(check_ptr(ctx, dL, "dL", nsub));
  CHECK_OK(check_ptr(ctx, dM, "dM", nsub));
  CHECK_OK(check_ptr(ctx, dmass, "dmass", nsub));
  if (ctx->adjoint_form == 1 && ctx->m2l_kernel == 1)
    return set_err(ctx, FMM_EINVAL, "the reference kernel computes the dense adjoint only");
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) return FMM_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  DescEntry* e = nullptr;
  const int need = ctx->m2l_kernel == 1 ? kNeedNone : need_adjoint(ctx->adjoint_form == 1);
  CHECK_OK(get_desc(ctx, desc, nsub, s, need, &e));
  const bool aligned = ((reinterpret_cast<uintptr_t>(pos) | reinterpret_cast<uintptr_t>(dmass)) & 15u) == 0;
  const bool harm = ctx->adjoint_form == 1;
  if (ctx->m2l_kernel != 1) CHECK_OK(ensure_lists(ctx, e, need_adjoint(harm), s));
  if (ctx->m2l_kernel != 1 && ppc == 8 && e->part_even && aligned && e->adjoint_plan[harm].fuse) {
    HIP_TRY(ctx, launch_m2l_mfma_backward(ctx->mfma, e->lists[need_adjoint(harm)].whole, e->d_desc, dL, dM, harm, s, pos, dmass));
  } else {
    if (ctx->m2l_kernel == 1) CHECK_OK(run_ref(ctx, e, true, dL, dM, s));
    else HIP_TRY(ctx, launch_m2l_mfma_backward(ctx->mfma, adjoint_list(e, harm), e->d_desc, dL, dM, harm, s));
    HIP_TRY(ctx, launch_p2m_backward(e->d_desc, nsub, e->d_ids, e->count, pos, ppc, dM, dmass, e->part_even, s));
  }
  return mark_used(ctx, e, s);
}

fmm_status fmm_stencil_tables(fmm_ctx* ctx, int32_t p, double* out, void* stream) {
  CHECK_OK(check_ctx(ctx));
  if (p < 2 || p > kMaxP) return set_err(ctx, FMM_EINVAL, "p not in {2,3,4}");
  CHECK_OK(check_ptr(ctx, out, "out", 1));
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  const int C = ncomp(p);
  HIP_TRY(ctx, hipMemcpyAsync(out, ctx->d_T[p], sizeof(double) * kNStencil * C * C,
                              hipMemcpyDeviceToDevice, static_cast<hipStream_t>(stream)));
  return FMM_OK;
}

fmm_status fmm_autotune(fmm_ctx* ctx, const fmm_subgrid* desc, int64_t nsub, const double* M,
                        double* L, fmm_precision prec, void* stream, int32_t* chosen) {
  CHECK_OK(check_ctx(ctx));
  CHECK_OK(check_desc(ctx, desc, nsub));
  CHECK_OK(check_ptr(ctx, M, "M", nsub));
  CHECK_OK(check_ptr(ctx, L, "L", nsub));
  CHECK_OK(check_precision(ctx, desc, nsub, prec));
  if (ctx->host_only) return set_err(ctx, FMM_EUNSUPPORTED, "host-only context");
  if (nsub == 0) {
    if (chosen) *chosen = pick_config(ctx, nullptr, prec);
    return FMM_OK;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  DeviceGuard guard(ctx->device);
  HIP_TRY(ctx, guard.err);
  DescEntry* e = nullptr;
  const int need = need_forward(prec == FMM_FP64_HARMONIC || prec == FMM_EXACT_SLICE);
  CHECK_OK(get_desc(ctx, desc, nsub, s, need, &e));
  if (prec == FMM_EXACT_SLICE) {
    // one kernel: nothing to time
    e->tuned[prec] = mfma_default_config(prec);
    if (chosen) *chosen = e->tuned[prec];
    return mark_used(ctx, e, s);
  }
  const bool harm = prec == FMM_FP64_HARMONIC;
  CHECK_OK(ensure_lists(ctx, e, need_forward(harm), s));
  WorkList per_wave = e->lists[need_forward(harm)].whole;
  per_wave.counter += 1;
  hipEvent_t t0, t1;
  HIP_TRY(ctx, hipEventCreate(&t0));
  HIP_TRY(ctx, hipEventCreate(&t1));
  int best = -1, best_parts = -1;   // the faster list of the streamed configurations (one kernel)
  float best_ms = 0.f, stream_ms = 0.f;
  for (int cfg = 0; cfg < mfma_num_configs(); ++cfg) {
    if (!mfma_config_supports(cfg, prec) || !mfma_config_distinct(cfg)) continue;
    const bool streams = mfma_config_streams(cfg);
    const CallLists& l = e->lists[need_forward(harm)];
    for (int parts = 0; parts < (streams && l.cut.count > 0 ? 2 : 1); ++parts) {
      // one warm-up launch, then the best of three
      auto launch = [&]() {
        return streams ? launch_m2l_stream(ctx->mfma, parts ? l.cut : l.whole, e->d_desc, M, L, harm, s)
               : prec == FMM_SPLIT_FP32 ? launch_m2l_split(ctx->mfma, l.whole, e->d_desc, M, L, s)
                                        : launch_m2l_mfma(ctx->mfma, per_wave, e->d_desc, M, L, prec, cfg, s);
      };
      HIP_TRY(ctx, launch());
      float ms = 1e30f;
      for (int r = 0; r < 3; ++r) {
        HIP_TRY(ctx, hipEventRecord(t0, s));
        HIP_TRY(ctx, launch());
        HIP_TRY(ctx, hipEventRecord(t1, s));
        HIP_TRY(ctx, hipEventSynchronize(t1));
        float one = 0.f;
        HIP_TRY(ctx, hipEventElapsedTime(&one, t0, t1));
        ms = std::min(ms, one);
      }
      if (best < 0 || ms < best_ms) {
        best = cfg;
        best_ms = ms;
      }
      if (streams && (parts == 0 || ms < stream_ms)) {
        best_parts = parts;
        stream_ms = ms;
      }
    }
  }
  (void)hipEventDestroy(t0);
  (void)hipEventDestroy(t1);
  e->tuned[prec] = best;
  e->tuned_parts[prec] = best_parts;
  if (chosen) *chosen = best;
  return mark_used(ctx, e, s);
}

}  // extern "C"
