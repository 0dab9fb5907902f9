// Entry points that keep host tables, with the host's memory running out at every allocation in
// turn: each call returns a status, and no exception leaves the library; what a plan asks of the
// device.  The HIP runtime
// calls and operator new are defined here (see check_flags.cpp).
//   no_memory <liblre.so>
#include <dlfcn.h>
#include <stdint.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <new>

#include "lre.h"

static int left = -1;           // allocations until one fails (-1: never)
static long device_blocks = 0;  // of hipMalloc, not yet freed
static long device_calls = 0;   // allocations, copies and waits

static void* take(size_t n) {
  if (left == 0) return nullptr;
  if (left > 0) --left;
  return std::malloc(n ? n : 1);
}
void* operator new(size_t n) {
  void* p = take(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return take(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
void operator delete(void* p, const std::nothrow_t&) noexcept { std::free(p); }

extern "C" {
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
int hipDeviceSynchronize() { ++device_calls; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipMalloc(void** p, size_t n) { ++device_calls; ++device_blocks; *p = std::calloc(1, n); return 0; }
int hipFree(void* p) { device_blocks -= p != nullptr; std::free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return 1; }
int hipMemcpy(void* dst, const void* src, size_t n, int) { ++device_calls; std::memcpy(dst, src, n); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = nullptr; return 0; }
}

int main(int argc, char** argv) {
  void* lib = argc > 1 ? dlopen(argv[1], RTLD_NOW | RTLD_LOCAL) : nullptr;
  if (!lib) return std::printf("%s\n", dlerror()), 2;
  auto create = reinterpret_cast<decltype(&lre_create)>(dlsym(lib, "lre_create"));
  auto plan = reinterpret_cast<decltype(&lre_batch_plan)>(dlsym(lib, "lre_batch_plan"));
  auto set_tiles = reinterpret_cast<decltype(&lre_batch_set_tiles)>(dlsym(lib, "lre_batch_set_tiles"));
  auto get_tiles = reinterpret_cast<decltype(&lre_batch_get_tiles)>(dlsym(lib, "lre_batch_get_tiles"));
  auto destroy = reinterpret_cast<decltype(&lre_batch_destroy)>(dlsym(lib, "lre_batch_destroy"));
  auto stream = reinterpret_cast<decltype(&lre_stream_create)>(dlsym(lib, "lre_stream_create"));
  auto stream_destroy = reinterpret_cast<decltype(&lre_stream_destroy)>(dlsym(lib, "lre_stream_destroy"));
  lre_ctx* ctx = nullptr;
  if (create(&ctx, 0) != LRE_OK) return 2;
  alignas(16) static char buffer[16];
  lre_instance inst[5];
  for (int j = 0; j < 5; ++j)
    inst[j] = lre_instance{5 + j, reinterpret_cast<uint16_t*>(buffer), (uint64_t)(j == 2 || j == 3 ? 0 : 20), nullptr,
                           reinterpret_cast<double*>(buffer), buffer};
  const long before = device_blocks;
  lre_batch* B = nullptr;
  int k = 0;
  for (; k < 10000; ++k) {
    left = k;
    const lre_status s = plan(ctx, inst, 5, 0, &B);
    left = -1;
    if (s == LRE_OK) break;
    if (s != LRE_E_HIP || B) return std::printf("plan, allocation %d fails: status %d\n", k, s), 1;
    if (device_blocks != before) return std::printf("plan, allocation %d fails: device memory kept\n", k), 1;
  }
  if (!B) return std::printf("no plan\n"), 1;
  // a plan is one allocation and one copy
  lre_batch* other = nullptr;
  device_calls = 0;
  if (plan(ctx, inst, 5, 0, &other) != LRE_OK || device_calls != 2)
    return std::printf("a plan takes %ld allocations, copies and waits\n", device_calls), 1;
  destroy(other);
  // the list is long enough for the smallest work items, in any mixture
  for (int first = 0; first < 5; ++first)
    for (int count = 1; first + count <= 5; ++count)
      for (unsigned flags : {0u, (unsigned)LRE_NO_RHO}) {
        const lre_batch_tiles least{1, 1, 432, 1, 1, 0};
        if (plan(ctx, inst + first, count, flags, &other) != LRE_OK || set_tiles(other, &least) != LRE_OK)
          return std::printf("work list of instances %d..%d\n", first, first + count - 1), 1;
        destroy(other);
      }
  lre_batch_tiles old{}, now{};
  get_tiles(B, &old, nullptr);
  const lre_batch_tiles list{1, 2, 432, 1, 0, 0};
  for (k = 0; k < 10000; ++k) {
    left = k;
    const lre_status s = set_tiles(B, &list);
    left = -1;
    get_tiles(B, &now, nullptr);
    if (s == LRE_OK) break;
    if (s != LRE_E_HIP) return std::printf("shape, allocation %d fails: status %d\n", k, s), 1;
    if (std::memcmp(&old, &now, sizeof old)) return std::printf("shape, allocation %d fails: shape changed\n", k), 1;
  }
  destroy(B);
  lre_stream* S = nullptr;
  for (k = 0; k < 10000; ++k) {
    left = k;
    const lre_status s = stream(ctx, 10, 2, 20, 0, &S);
    left = -1;
    if (s == LRE_OK) break;
    if (s != LRE_E_HIP || S) return std::printf("stream, allocation %d fails: status %d\n", k, s), 1;
  }
  stream_destroy(S);
  return device_blocks == before ? 0 : (std::printf("device memory kept\n"), 1);
}
