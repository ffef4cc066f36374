// A HIP runtime of ordinary memory, and a tile kernel of one token per byte, for
// tests of the host code (tt_api.hip, tt_session.hip) on the CPU: which memory a
// call takes, what it does when there is none, and what it hands to the kernel.
//
// Device and pinned memory have budgets (fake_budgets).  As with the runtime
// itself, the last error stays until it is read.  The "kernel" ends the process
// when it is given memory that a device could not reach.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>

#include "tt_internal.h"

using namespace tt;

namespace {

struct Block {
  size_t n;
  bool pinned;
};
std::mutex mu;
std::map<uintptr_t, Block> blocks;
size_t used[2], budget[2] = {SIZE_MAX, SIZE_MAX};  // device, pinned
thread_local hipError_t last = hipSuccess;
int32_t documents;  // of the last batch, as the kernel got them

hipError_t fail(hipError_t e) { return last = e; }

hipError_t take(void** p, size_t n, bool pinned) {
  std::lock_guard<std::mutex> g(mu);
  if (n > budget[pinned] || used[pinned] > budget[pinned] - n) return fail(hipErrorOutOfMemory);
  *p = malloc(n ? n : 1);
  memset(*p, 0xA5, n);
  used[pinned] += n;
  blocks[(uintptr_t)*p] = Block{n, pinned};
  return hipSuccess;
}

hipError_t give(void* p, bool pinned) {
  std::lock_guard<std::mutex> g(mu);
  auto it = blocks.find((uintptr_t)p);
  if (it == blocks.end() || it->second.pinned != pinned) abort();
  used[pinned] -= it->second.n;
  blocks.erase(it);
  free(p);
  return hipSuccess;
}

const Block* block_of(const void* p, size_t n) {
  std::lock_guard<std::mutex> g(mu);
  auto it = blocks.upper_bound((uintptr_t)p);
  if (it == blocks.begin()) return nullptr;
  --it;
  return (uintptr_t)p + n <= it->first + it->second.n ? &it->second : nullptr;
}

void reach(const void* p, size_t n, const char* what) {
  if (n != 0 && !block_of(p, n)) {
    fprintf(stderr, "the device cannot reach %s\n", what);
    abort();
  }
}

bool valid(const uint8_t* s, int64_t n) {
  for (int64_t i = 0; i < n;) {
    const int l = s[i] < 0x80 ? 1 : s[i] < 0xC2 ? 0 : s[i] < 0xE0 ? 2 : s[i] < 0xF0 ? 3 : s[i] < 0xF5 ? 4 : 0;
    if (l == 0 || i + l > n) return false;
    for (int k = 1; k < l; ++k)
      if ((s[i + k] & 0xC0) != 0x80) return false;
    i += l;
  }
  return true;
}

}  // namespace

hipError_t hipMalloc(void** p, size_t n) { return take(p, n, false); }
hipError_t hipFree(void* p) { return give(p, false); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return take(p, n, true); }
hipError_t hipHostFree(void* p) { return give(p, true); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
  reach(k == hipMemcpyHostToDevice ? d : s, n, "a copy's device side");
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  reach(d, n, "a fill's memory");
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  const Block* b = block_of(p, 1);
  if (!b) return fail(hipErrorInvalidValue);
  a->type = b->pinned ? hipMemoryTypeHost : hipMemoryTypeDevice;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}

namespace {

void kernel(Work w, DevTables tb, int mode) {
  const int64_t n = w.n;
  // (a tile waits for ever when the tiles before it have the tickets of another call)
  if (w.ctrl->tile_ticket != w.ticket_base) {
    fprintf(stderr, "the call's tickets begin at %u, the counter stands at %u\n", w.ticket_base, w.ctrl->tile_ticket);
    abort();
  }
  w.ctrl->tile_ticket += w.n_tiles;
  reach(w.text, (size_t)n, "the request");
  reach(w.out_len, 8, "the output length");
  bool ok = valid(w.text, n);
  if (w.doc_off) {
    documents = w.n_docs;
    const size_t nd = (size_t)w.n_docs + 1;
    reach(w.doc_off, 8 * nd, "the document offsets");
    reach(w.out_doc_off, 8 * nd, "the output offsets");
    reach(w.tile_docs, 8 * (size_t)w.n_tiles, "the tiles' documents");
    for (size_t d = 0; d + 1 < nd; ++d) ok = ok && valid(w.text + w.doc_off[d], w.doc_off[d + 1] - w.doc_off[d]);
    for (uint32_t t = 0; t < w.n_tiles; ++t) {
      const int64_t lo = (int64_t)t * PT_OWN - PT_HALO - PT_PAD, hi = (int64_t)t * PT_OWN - PT_HALO + PT_WIN;
      const uint2 x = w.tile_docs[t];
      if ((x.x > 0 && w.doc_off[x.x - 1] >= lo) || (x.x < (uint32_t)w.n_docs && w.doc_off[x.x] < lo) ||
          (x.y > 0 && w.doc_off[x.y - 1] >= hi) || (x.y < (uint32_t)w.n_docs && w.doc_off[x.y] < hi)) {
        fprintf(stderr, "tile %u has documents [%u, %u)\n", t, x.x, x.y);
        abort();
      }
    }
    for (size_t d = 0; d < nd; ++d)
      w.out_doc_off[d] = !ok && w.doc_off[d] >= n ? (int64_t)TT_ERR_INVALID_UTF8 : w.doc_off[d];
  }
  *w.out_len = ok ? n : (int64_t)TT_ERR_INVALID_UTF8;
  if (w.out16) reach(w.out16, 2 * (size_t)n, "the 16-bit IDs");
  else reach(w.out_ids, 4 * (size_t)n, "the IDs");
  if (w.out_hi) reach(w.out_hi, (size_t)n, "the IDs' third bytes");
  if (mode == 2) reach(w.out_spans, 16 * (size_t)n, "the spans");
  int32_t chars = 0;
  for (int64_t i = 0; i < n; ++i) {
    const uint32_t id = (uint32_t)tb.ext_id[w.text[i]];
    chars += (w.text[i] & 0xC0) != 0x80;
    if (w.out16) w.out16[i] = (uint16_t)id;
    else w.out_ids[i] = mode == 0 ? (int32_t)i : (int32_t)id;
    if (w.out_hi) w.out_hi[i] = (uint8_t)(id >> 16);
    if (mode == 2) {
      const int32_t s[4] = {(int32_t)i, (int32_t)i + 1, chars - 1, chars};
      memcpy(w.out_spans + 4 * i, s, 16);
    }
  }
}

}  // namespace

// (the library's launches report their own status, whatever the last error is)
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  if (f != reinterpret_cast<const void*>(&kernel)) abort();
  kernel(*static_cast<Work*>(args[0]), *static_cast<DevTables*>(args[1]), *static_cast<int*>(args[2]));
  return hipSuccess;
}

namespace tt {
hipError_t launch_tile(const Work& w, const DevTables& tb, int, int mode, bool, hipStream_t s) {
  return launch(kernel, dim3(w.n_tiles), dim3(PT_THREADS), s, w, tb, mode);
}
}  // namespace tt


// What device and pinned allocations may hold in all (bytes).
extern "C" void fake_budgets(uint64_t device, uint64_t pinned) {
  budget[0] = device;
  budget[1] = pinned;
}
extern "C" uint64_t fake_used(int pinned) { return used[pinned]; }
extern "C" int fake_last_error() { return (int)hipGetLastError(); }
extern "C" void* fake_device(uint64_t n) {
  void* p = nullptr;
  return hipMalloc(&p, (size_t)n) == hipSuccess ? p : nullptr;
}
extern "C" void fake_free(void* p) { (void)hipFree(p); }
extern "C" int32_t fake_documents() { return documents; }
