// Error reporting, device check, handle bookkeeping and the host-side
// evaluation of the classification predicates.
#include <string.h>

#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "geometry.h"
#include "internal.h"

namespace {
thread_local char g_last_hip[256] = "";
std::mutex g_dev_mu;
int g_dev_ok[64];  // 0 unknown, 1 gfx950, 2 other

struct Block {
  char* p;
  size_t bytes;
  uint64_t stamp;
};
struct DevicePool {
  std::vector<Block> blocks;
  std::vector<int64_t*> pinned;
  size_t bytes = 0;
  uint64_t gives = 0;
  void* anchor = nullptr;  // see handle_idle
};
// never destroyed: the runtime may be gone before this object would be
struct Pools {
  std::mutex mu;
  DevicePool dev[64];
};
Pools* pools() {
  static Pools* p = new (std::nothrow) Pools();
  return p;
}

// frees on device dev, from whatever device is current
template <typename F>
void on_device(int dev, F f) {
  int cur = dev;
  (void)hipGetDevice(&cur);
  if (cur != dev) (void)hipSetDevice(dev);
  f();
  if (cur != dev) (void)hipSetDevice(cur);
}

// allocations and frees of its scope leave another thread's stream capture alone
struct CaptureRelaxed {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  bool on = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  ~CaptureRelaxed() {
    if (on) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

}  // namespace

namespace csc {

void pool_empty(int dev) {
  if (!pools() || dev < 0 || dev >= 64) return;
  std::vector<Block> all;
  std::vector<int64_t*> words;
  {
    std::lock_guard<std::mutex> lk(pools()->mu);
    all.swap(pools()->dev[dev].blocks);
    words.swap(pools()->dev[dev].pinned);
    pools()->dev[dev].bytes = 0;
  }
  CaptureRelaxed relaxed;
  for (const Block& b : all) (void)hipFree(b.p);
  for (int64_t* w : words) (void)hipHostFree(w);
}

hipError_t device_alloc(size_t bytes, void** p, int dev) {
  CaptureRelaxed relaxed;
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    pool_empty(dev);
    e = hipMalloc(p, bytes);
  }
  if (e != hipSuccess) *p = nullptr;
  return e;
}

int fail_hip(hipError_t e) {
  const char* s = hipGetErrorString(e);
  strncpy(g_last_hip, s ? s : "unknown HIP error", sizeof(g_last_hip) - 1);
  g_last_hip[sizeof(g_last_hip) - 1] = 0;
  return CSC_HIP_ERROR;
}

int check_device() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e);
  if (dev < 0 || dev >= 64) return CSC_UNSUPPORTED_DEVICE;
  std::lock_guard<std::mutex> lk(g_dev_mu);
  if (g_dev_ok[dev] == 0) {
    hipDeviceProp_t p;
    e = hipGetDeviceProperties(&p, dev);
    if (e != hipSuccess) return fail_hip(e);
    g_dev_ok[dev] = strncmp(p.gcnArchName, "gfx950", 6) == 0 ? 1 : 2;
  }
  return g_dev_ok[dev] == 1 ? CSC_OK : CSC_UNSUPPORTED_DEVICE;
}

hipError_t pool_take(size_t bytes, char** p, size_t* got, int* dev) {
  hipError_t e = hipGetDevice(dev);
  if (e != hipSuccess) return e;
  const bool pooled = pools() && *dev >= 0 && *dev < 64;
  if (pooled) {
    std::lock_guard<std::mutex> lk(pools()->mu);
    DevicePool& D = pools()->dev[*dev];
    // the smallest that holds it, unless more than half of it would lie idle
    const size_t most = bytes > ((size_t)1 << 20) ? 2 * bytes : (size_t)2 << 20;
    int best = -1;
    for (int i = 0; i < (int)D.blocks.size(); i++)
      if (D.blocks[i].bytes >= bytes && D.blocks[i].bytes <= most &&
          (best < 0 || D.blocks[i].bytes < D.blocks[best].bytes))
        best = i;
    if (best >= 0) {
      *p = D.blocks[best].p;
      *got = D.blocks[best].bytes;
      D.bytes -= D.blocks[best].bytes;
      D.blocks[best] = D.blocks.back();
      D.blocks.pop_back();
      return hipSuccess;
    }
  }
  CaptureRelaxed relaxed;
  // up to an eighth more, so that the block serves a somewhat larger mesh as well
  size_t step = 4096;
  while (step * 16 <= bytes) step *= 2;
  const size_t round = pooled ? (bytes + step - 1) / step * step : bytes;
  if (round > bytes) {  // without the rounding where that does not fit
    e = hipMalloc((void**)p, round);
    *got = round;
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
  }
  *got = bytes;
  return device_alloc(bytes, (void**)p, *dev);
}

void pool_give(int dev, char* p, size_t bytes) {
  std::vector<Block> old;
  if (pools() && dev >= 0 && dev < 64 && bytes <= POOL_BYTES) {
    try {
      std::lock_guard<std::mutex> lk(pools()->mu);
      DevicePool& D = pools()->dev[dev];
      D.gives++;
      old.reserve(D.blocks.size());
      D.blocks.reserve(POOL_BLOCKS + 1);
      D.blocks.push_back(Block{p, bytes, D.gives});
      D.bytes += bytes;
      p = nullptr;
      // out: the unused, and the oldest while there are too many
      for (size_t i = 0; i < D.blocks.size();) {
        size_t oldest = 0;
        for (size_t j = 1; j < D.blocks.size(); j++)
          if (D.blocks[j].stamp < D.blocks[oldest].stamp) oldest = j;
        if (D.bytes <= POOL_BYTES && D.blocks.size() <= POOL_BLOCKS && D.gives - D.blocks[oldest].stamp <= POOL_AGE)
          break;
        old.push_back(D.blocks[oldest]);
        D.bytes -= D.blocks[oldest].bytes;
        D.blocks[oldest] = D.blocks.back();
        D.blocks.pop_back();
      }
    } catch (const std::bad_alloc&) {  // p is not kept then
    }
  }
  if (!p && old.empty()) return;
  CaptureRelaxed relaxed;
  if (p) (void)hipFree(p);
  for (const Block& b : old) (void)hipFree(b.p);
}

hipError_t pinned_take(int64_t** p, int* dev) {
  hipError_t e = hipGetDevice(dev);
  if (e != hipSuccess) return e;
  if (pools() && *dev >= 0 && *dev < 64) {
    std::lock_guard<std::mutex> lk(pools()->mu);
    std::vector<int64_t*>& v = pools()->dev[*dev].pinned;
    if (!v.empty()) {
      *p = v.back();
      v.pop_back();
      return hipSuccess;
    }
  }
  CaptureRelaxed relaxed;
  e = hipHostMalloc((void**)p, sizeof(int64_t) * PINNED_WORDS, hipHostMallocDefault);
  if (e != hipSuccess) *p = nullptr;
  return e;
}

void pinned_give(int dev, int64_t* p) {
  if (pools() && dev >= 0 && dev < 64) {
    try {
      std::lock_guard<std::mutex> lk(pools()->mu);
      std::vector<int64_t*>& v = pools()->dev[dev].pinned;
      if (v.size() < (size_t)POOL_BLOCKS) {
        v.push_back(p);
        return;
      }
    } catch (const std::bad_alloc&) {
    }
  }
  CaptureRelaxed relaxed;
  (void)hipHostFree(p);
}

// Waits for the work queued on a handle. Allowed in every capture mode of the calling
// thread and of others: hipDeviceSynchronize is refused while any thread captures, and
// ends that capture. A handle used on the null stream alone waits for that one. Otherwise
// hipFree waits for the whole device (its streams may be gone by now); an allocation of a
// few bytes is freed for that. It also writes the L2 back: 12 to 40 us more than the null
// stream's wait after a field of 1 to 42 MB. (20 more where the allocation is the only
// one of its size, since the runtime then maps and unmaps its page each time: one such allocation per device
// is kept.)
bool handle_idle(const csc_features* f) {
  CaptureRelaxed relaxed;
  bool idle = false;
  const int dev = f->device;
  on_device(dev, [&] {
    if (!f->other_streams.load(std::memory_order_relaxed)) {
      idle = hipStreamSynchronize(nullptr) == hipSuccess;
      if (idle) return;
      (void)hipGetLastError();
    }
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, 64);
    if (e == hipSuccess && pools() && dev >= 0 && dev < 64) {
      std::lock_guard<std::mutex> lk(pools()->mu);
      if (!pools()->dev[dev].anchor) std::swap(pools()->dev[dev].anchor, p);
    }
    if (e == hipSuccess && !p) e = hipMalloc(&p, 64);
    if (e == hipSuccess) idle = hipFree(p) == hipSuccess;
    else (void)hipGetLastError();
  });
  return idle;
}

}  // namespace csc

using namespace csc;

extern "C" const char* csc_error_string(int code) {
  switch (code) {
    case CSC_OK: return "ok";
    case CSC_INVALID_ARG: return "invalid argument";
    case CSC_NONMANIFOLD: return "surface is open or non-manifold (an edge without exactly two triangles)";
    case CSC_INCONSISTENT_ORIENTATION: return "inconsistent orientation (a directed edge occurs twice)";
    case CSC_DEGENERATE_FACE: return "degenerate (zero-area) triangle";
    case CSC_GRID_TOO_LARGE: return "grid too large";
    case CSC_OUT_OF_MEMORY: return "out of device memory";
    case CSC_HIP_ERROR: return "HIP runtime error";
    case CSC_WORKSPACE_TOO_SMALL: return "workspace too small";
    case CSC_UNSUPPORTED_DEVICE: return "unsupported device (gfx950 required)";
    default: return "unknown status";
  }
}

extern "C" const char* csc_last_hip_error(void) { return g_last_hip; }

extern "C" int csc_features_info(const csc_features* f, csc_feature_info* info) {
  if (!f || !f->synced || !info) return CSC_INVALID_ARG;
  *info = f->info;
  return CSC_OK;
}

extern "C" void csc_features_free(csc_features* f) {
  if (!f) return;
  // What the handle queued may still run, on any stream: its memory is kept for the
  // next handle only once the device has finished it (as hipFree would wait for it).
  CaptureRelaxed relaxed;  // a handle may be freed while another thread, or this one, captures
  const bool idle = (f->arena || f->h_stats) && handle_idle(f);
  if (f->arena) {
    if (idle) pool_give(f->device, f->arena, f->arena_bytes);
    else (void)hipFree(f->arena);
  }
  if (f->face_order) (void)hipFree(f->face_order);
  if (f->h_stats) {
    if (idle) pinned_give(f->device, f->h_stats);
    else (void)hipHostFree(f->h_stats);
  }
  delete f;
}

extern "C" void csc_release_memory(void) {
  int devices = 0;
  if (hipGetDeviceCount(&devices) != hipSuccess) return;
  for (int dev = 0; dev < devices; dev++) pool_empty(dev);
}

extern "C" int csc_classify_edge(const float a[3], const float b[3], const float c1[3], const float c2[3]) {
  if (!a || !b || !c1 || !c2) return -CSC_INVALID_ARG;
  return classify_edge(mk(a[0], a[1], a[2]), mk(b[0], b[1], b[2]), mk(c1[0], c1[1], c1[2]), mk(c2[0], c2[1], c2[2]));
}

extern "C" int csc_classify_vertex(const float v[3], const float* ring, int32_t n_faces, const csc_options* opt,
                                   double axis[3], double* cos_t) {
  if (!v || !ring || n_faces <= 0 || !axis || !cos_t) return -CSC_INVALID_ARG;
  csc_options o = {1e-3f, 0, 0, 0, {0, 0, 0}, 0, 0.f, 0, 0, 0};
  if (opt) o = *opt;
  d3 pv = mkd(v[0], v[1], v[2]);
  VertexAccum acc;
  for (int i = 0; i < n_faces; i++) {
    const float* p = ring + 6 * i;
    acc.add_face(pv, mkd(p[0], p[1], p[2]), mkd(p[3], p[4], p[5]));
  }
  VertexTest t;
  t.init(acc.n_alpha);
  for (int i = 0; i < n_faces; i++) {
    const float* p = ring + 6 * i;
    d3 p1 = mkd(p[0], p[1], p[2]), p2 = mkd(p[3], p[4], p[5]);
    t.neighbour(pv, p1);
    t.normal(pv, p1, p2);
  }
  VertexClass vc = t.finish(o.ruff_mode, o.saddle_mode, o.force_both_sides);
  axis[0] = vc.axis.x;
  axis[1] = vc.axis.y;
  axis[2] = vc.axis.z;
  *cos_t = vc.cos_t;
  return (int)vc.bits;
}
