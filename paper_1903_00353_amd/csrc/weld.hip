// Triangle-soup ingestion (Section 7, Section 7.1-7.2): an STL file lists every
// triangle with its own three corner positions, so a vertex shared by k
// triangles appears k times. Welding gives every distinct position one vertex
// index, turning the soup into the indexed mesh the feature build reads; the
// edge pairs then follow from the indexed mesh (twins around each vertex).
//
// The paper orders corners by 30-bit Morton codes, which can map different
// positions to the same code and leave a per-group sequential pass to separate
// them. Here the corners meet in a hash table keyed by their exact position (-0
// taken as +0 first: equal as positions), whose entry becomes the smallest corner
// of the position: nothing is ordered, and nothing is left to sort out per group.
// Vertices are numbered in order of first appearance in the soup: a prefix sum
// over the corners that are the smallest of their position.
//
// What bounds it: the table's scattered accesses (one line of the table and one of
// the soup per corner). Five launches; ordering the corners by three stable 32-bit
// radix sorts instead took 61 (1.08M corners: 532 -> 170 us a call, 75 of it on the device; 15.7M
// corners: 3.75 -> 1.03 ms).
#include <cmath>
#include <mutex>

#include "internal.h"
#include "wave.h"

namespace csc {

constexpr int32_t WELD_EMPTY = INT32_MAX;  // above every corner index
constexpr int WB = 256, WITEMS = 8, WTILE = WB * WITEMS;
constexpr int64_t WELD_SHORT_TILES = 4096;

// slots of the table for n corners: at most two thirds full
__host__ __device__ inline int64_t weld_slots(int64_t n) { return n + n / 2 + 64; }

struct WeldKey {
  uint32_t x, y, z;
  __device__ bool operator==(const WeldKey& o) const { return x == o.x && y == o.y && z == o.z; }
};

// the position bits of a corner, -0 mapped to +0
__device__ inline WeldKey weld_key(const float* __restrict__ soup, int64_t c) {
  const float x = soup[3 * c], y = soup[3 * c + 1], z = soup[3 * c + 2];
  return WeldKey{__float_as_uint(x == 0.f ? 0.f : x), __float_as_uint(y == 0.f ? 0.f : y),
                 __float_as_uint(z == 0.f ? 0.f : z)};
}

__device__ inline bool finite_bits(uint32_t b) { return (b & 0x7f800000u) != 0x7f800000u; }

// A 32-bit mix of the three words: the final avalanche of xxHash32 (Y. Collet; its shifts
// and its prime multipliers) with a word added before each of its multiplications, and
// one more of its primes. Keys of grids of 128^3 to 200^3 points, whole numbers or
// fractions, lie at most 20 slots from their own in a table of single corners, symmetric ones 29.
__device__ inline uint32_t weld_hash(const WeldKey& k) {
  uint32_t h = k.x * 0x9e3779b1u;
  h = (h ^ (h >> 15) ^ k.y) * 0x85ebca77u;
  h = (h ^ (h >> 13) ^ k.z) * 0xc2b2ae3du;
  h = (h ^ (h >> 16)) * 0x27d4eb2fu;
  return h ^ (h >> 15);
}

// every slot empty; the flag and count words cleared
__global__ void k_weld_clear(int32_t* table, int64_t slots, int32_t* bad) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i == 0) *bad = 0;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = i; k < slots; k += step) table[k] = WELD_EMPTY;
}

// Every corner finds its position's slot (linear probing from its hash) and leaves
// there the smaller of itself and the corner it meets; a slot once claimed keeps its
// position, so the comparison may read any corner it held. A corner that sees a
// smaller one of its position adds nothing: many equal corners cost one atomic, not
// one each. The table holds at least n / 2 empty slots, so every search ends.
__global__ __launch_bounds__(WB) void k_weld_insert(const float* __restrict__ soup, int64_t n, int64_t slots,
                                                    int32_t* table, uint32_t* slot_of, int32_t* bad) {
  const int64_t c = blockIdx.x * (int64_t)WB + threadIdx.x;
  if (c >= n) return;
  const WeldKey k = weld_key(soup, c);
  if (!finite_bits(k.x) || !finite_bits(k.y) || !finite_bits(k.z)) *bad = 1;
  int64_t h = (int64_t)(((uint64_t)weld_hash(k) * (uint64_t)slots) >> 32);
  for (;;) {
    int32_t at = __hip_atomic_load(&table[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (at == WELD_EMPTY) {
      at = atomicCAS(&table[h], WELD_EMPTY, (int32_t)c);
      if (at == WELD_EMPTY) break;  // claimed
    }
    if (weld_key(soup, at) == k) {
      if (at > (int32_t)c) atomicMin(&table[h], (int32_t)c);
      break;
    }
    if (++h == slots) h = 0;
  }
  slot_of[c] = (uint32_t)h;
}

// every corner's first corner (in place of its slot), and the number of first
// corners in each tile
__global__ __launch_bounds__(WB) void k_weld_first(const int32_t* __restrict__ table, int64_t n, uint32_t* slot_of,
                                                   int32_t* sums) {
  __shared__ int ws[WB / 64];
  const int64_t base = (int64_t)blockIdx.x * WTILE;
  int heads = 0;
#pragma unroll
  for (int i = 0; i < WITEMS; i++) {
    const int64_t c = base + i * WB + threadIdx.x;
    int32_t f = -1;
    if (c < n) {
      f = table[slot_of[c]];
      slot_of[c] = (uint32_t)f;
    }
    heads += __popcll(__ballot(c < n && f == (int32_t)c));
  }
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = heads;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < WB / 64; w++) t += ws[w];
    sums[blockIdx.x] = t;
  }
}

// the vertex number of every first corner (its rank in corner order) and that
// vertex's position; the tile's offset is the sum of the tile counts before it,
// added up by the block itself when the tiles are few (scanned beforehand if not)
__global__ __launch_bounds__(WB) void k_weld_vertices(const float* __restrict__ soup, int64_t n,
                                                      const uint32_t* __restrict__ first,
                                                      const int32_t* __restrict__ sums, int scanned, int32_t* vid,
                                                      float* verts, int64_t* total) {
  __shared__ int ws[WB / 64], wh[WITEMS][WB / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int pre = 0;
  if (!scanned)
    for (int j = threadIdx.x; j < (int)blockIdx.x; j += WB) pre += sums[j];
  for (int o = 32; o > 0; o >>= 1) pre += __shfl_down(pre, o, 64);
  if (lane == 0) ws[w] = pre;
  const int64_t base = (int64_t)blockIdx.x * WTILE;
  unsigned long long m[WITEMS];
#pragma unroll
  for (int i = 0; i < WITEMS; i++) {
    const int64_t c = base + i * WB + threadIdx.x;
    m[i] = __ballot(c < n && first[c < n ? c : 0] == (uint32_t)c);
    if (lane == 0) wh[i][w] = __popcll(m[i]);
  }
  __syncthreads();
  int at = scanned ? sums[blockIdx.x] : 0;
  if (!scanned)
    for (int u = 0; u < WB / 64; u++) at += ws[u];
#pragma unroll
  for (int i = 0; i < WITEMS; i++) {
    int here = at;
    for (int u = 0; u < WB / 64; u++) {
      here += u < w ? wh[i][u] : 0;
      at += wh[i][u];
    }
    if ((m[i] >> lane) & 1) {
      const int64_t c = base + i * WB + threadIdx.x;
      const int64_t v = here + __popcll(m[i] & ((1ull << lane) - 1));
      vid[c] = (int32_t)v;
      verts[3 * v] = soup[3 * c];
      verts[3 * v + 1] = soup[3 * c + 1];
      verts[3 * v + 2] = soup[3 * c + 2];
    }
  }
  if (!scanned && threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) *total = at;
}

// every corner gets the vertex of its first corner
__global__ void k_weld_tris(const uint32_t* __restrict__ first, const int32_t* __restrict__ vid, int64_t n,
                            int32_t* tris) {
  const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (c < n) tris[c] = vid[first[c]];
}

}  // namespace csc

using namespace csc;

namespace {

// what a weld reports: read back with one copy
struct WeldCount {
  int64_t nv;
  int32_t bad, pad;
};

// scratch of a weld of n corners: the table, the corners' slots (then first
// corners), vertex numbers, tile counts, the report
struct WeldLayout {
  size_t slot, vid, sums, count, total;
};

WeldLayout weld_layout(int64_t n) {
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  WeldLayout L;
  L.slot = al(sizeof(int32_t) * (size_t)weld_slots(n));
  L.vid = L.slot + al(sizeof(uint32_t) * (size_t)n);
  L.sums = L.vid + al(sizeof(int32_t) * (size_t)n);
  L.count = L.sums + al(sizeof(int32_t) * (size_t)((n + WTILE - 1) / WTILE));
  L.total = L.count + al(sizeof(WeldCount));
  return L;
}

// the weld on scratch memory W (weld_layout(3 nf).total bytes); queues the
// kernels and the copy of the report on s, without synchronising
hipError_t weld_queue(const float* soup_d, int64_t nf, float* verts_d, int32_t* tris_d, char* W, const WeldLayout& L,
                      WeldCount* h, hipStream_t s) {
  const int64_t n = 3 * nf, slots = weld_slots(n), tiles = (n + WTILE - 1) / WTILE;
  int32_t* table = (int32_t*)W;
  uint32_t* slot = (uint32_t*)(W + L.slot);
  int32_t *vid = (int32_t*)(W + L.vid), *sums = (int32_t*)(W + L.sums);
  WeldCount* count = (WeldCount*)(W + L.count);
  hipError_t e;
  const unsigned fill = grid_1d(slots, 4 * WB);
  k_weld_clear<<<fill < 8192 ? fill : 8192, WB, 0, s>>>(table, slots, &count->bad);
  k_weld_insert<<<grid_1d(n, WB), WB, 0, s>>>(soup_d, n, slots, table, slot, &count->bad);
  k_weld_first<<<(unsigned)tiles, WB, 0, s>>>(table, n, slot, sums);
  const bool few = tiles <= WELD_SHORT_TILES;
  if (!few && (e = scan_sums_inplace(sums, tiles, &count->nv, s)) != hipSuccess) return e;
  k_weld_vertices<<<(unsigned)tiles, WB, 0, s>>>(soup_d, n, slot, sums, few ? 0 : 1, vid, verts_d, &count->nv);
  k_weld_tris<<<grid_1d(n, WB), WB, 0, s>>>(slot, vid, n, tris_d);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return hipMemcpyAsync(h, count, sizeof(WeldCount), hipMemcpyDeviceToHost, s);
}

bool weld_args_ok(const float* soup_d, int64_t nf, const float* verts_d, const int32_t* tris_d, const int64_t* nv) {
  return soup_d && verts_d && tris_d && nv && nf > 0 && 3 * nf < INT32_MAX;
}

}  // namespace

extern "C" int csc_weld_soup(const float* soup_d, int64_t nf, float* verts_d, int32_t* tris_d, int64_t* nv,
                             void* stream) {
  if (!weld_args_ok(soup_d, nf, verts_d, tris_d, nv)) return CSC_INVALID_ARG;
  int rc = check_device();
  if (rc != CSC_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  // the call synchronises s: refused while s is captured, before scratch is taken
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t ce = hipStreamIsCapturing(s, &cap);
  if (ce == hipSuccess && cap != hipStreamCaptureStatusNone) ce = hipErrorStreamCaptureUnsupported;
  if (ce != hipSuccess) return fail_hip(ce);
  const WeldLayout L = weld_layout(3 * nf);
  char* W = nullptr;
  int64_t* pinned = nullptr;
  size_t bytes = 0;
  int dev = 0;
  // scratch too large to be kept comes and goes on the stream: its free waits for
  // nobody else's work
  const bool keep = L.total <= POOL_BYTES;
  hipError_t e;
  if (keep) {
    e = pool_take(L.total, &W, &bytes, &dev);
  } else {
    e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipMallocAsync((void**)&W, L.total, s);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      pool_empty(dev);
      e = hipMallocAsync((void**)&W, L.total, s);
    }
  }
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? CSC_OUT_OF_MEMORY : fail_hip(e);
  e = pinned_take(&pinned, &dev);
  static_assert(sizeof(WeldCount) <= sizeof(int64_t) * PINNED_WORDS, "the report fits the pinned words");
  if (e == hipSuccess) e = weld_queue(soup_d, nf, verts_d, tris_d, W, L, (WeldCount*)pinned, s);
  if (!keep) {
    const hipError_t ef = hipFreeAsync(W, s);
    if (e == hipSuccess) e = ef;
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {  // queued work may still use them: freed, which waits for it
    if (keep) (void)hipFree(W);
    if (pinned) (void)hipHostFree(pinned);
    return fail_hip(e);
  }
  const WeldCount h = *(const WeldCount*)pinned;
  if (keep) pool_give(dev, W, bytes);
  pinned_give(dev, pinned);
  if (h.bad) return CSC_INVALID_ARG;
  *nv = h.nv;
  return CSC_OK;
}

// ------------------------------------------------------------ allocation-free
// csc_weld_soup_noalloc keeps its scratch in this file-scope device array, one
// copy per GPU, held until the process ends. Host code never passes the array's
// name to a kernel (on the host it only names the symbol): each device's
// address comes from hipGetSymbolAddress on the first call with that device
// current, and is kept per device.
constexpr size_t WELD_SCRATCH_BYTES = (size_t)64 << 20;
constexpr int64_t WELD_NOALLOC_FACES = 428096;  // the documented limit; their scratch takes 18 MB
static __device__ __align__(256) char scratch[WELD_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[MAX_DEVICES] = {};

int scratch_for_current_device(char** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e);
  if (dev < 0 || dev >= MAX_DEVICES) return CSC_UNSUPPORTED_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail_hip(e != hipSuccess ? e : hipErrorInvalidSymbol);
    g_scratch_ptr[dev] = (char*)p;
  }
  *out = g_scratch_ptr[dev];
  return CSC_OK;
}
}  // namespace

extern "C" int csc_weld_soup_noalloc(const float* soup_d, int64_t nf, float* verts_d, int32_t* tris_d, int64_t* nv,
                                     void* stream) {
  if (!weld_args_ok(soup_d, nf, verts_d, tris_d, nv)) return CSC_INVALID_ARG;
  if (nf > WELD_NOALLOC_FACES) return CSC_WORKSPACE_TOO_SMALL;
  const WeldLayout L = weld_layout(3 * nf);
  if (L.total > WELD_SCRATCH_BYTES) return CSC_WORKSPACE_TOO_SMALL;
  int rc = check_device();
  if (rc != CSC_OK) return rc;
  char* W = nullptr;
  rc = scratch_for_current_device(&W);
  if (rc != CSC_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  WeldCount h = {0, 0, 0};
  hipError_t e = weld_queue(soup_d, nf, verts_d, tris_d, W, L, &h, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail_hip(e);
  if (h.bad) return CSC_INVALID_ARG;
  *nv = h.nv;
  return CSC_OK;
}

extern "C" int64_t csc_weld_soup_noalloc_max_faces(void) { return WELD_NOALLOC_FACES; }
