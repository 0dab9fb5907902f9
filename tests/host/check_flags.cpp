// lre_check against a host that fails its copies: the HIP runtime calls of lre_create and lre_check
// are defined here (the library's references bind to the program's definitions), with host
// memory for device memory.
//   check_flags <liblre.so>
#include <dlfcn.h>
#include <stdint.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "lre.h"

namespace {
std::vector<void*> blocks;      // of hipMalloc
uint32_t* mirror = nullptr;     // of hipHostMalloc
int copies = 0, fail_copy = 0;  // copies so far; the one that fails (1, 2, ...)
}  // namespace

extern "C" {
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
int hipMalloc(void** p, size_t n) { blocks.push_back(*p = std::calloc(1, n)); return 0; }
int hipFree(void*) { return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { mirror = static_cast<uint32_t*>(*p = std::calloc(1, n)); return 0; }
int hipHostFree(void*) { return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return 1; }
int hipStreamSynchronize(void*) { return 0; }
int hipMemcpy(void* dst, const void* src, size_t n, int) {
  if (++copies == fail_copy) return 900;
  std::memcpy(dst, src, n);
  return 0;
}
}

int main(int argc, char** argv) {
  void* lib = argc > 1 ? dlopen(argv[1], RTLD_NOW | RTLD_LOCAL) : nullptr;
  if (!lib) return std::printf("%s\n", dlerror()), 2;
  auto create = reinterpret_cast<lre_status (*)(lre_ctx**, int)>(dlsym(lib, "lre_create"));
  auto check = reinterpret_cast<lre_status (*)(lre_ctx*, void*)>(dlsym(lib, "lre_check"));
  lre_ctx* ctx = nullptr;
  if (create(&ctx, 0) != LRE_OK || blocks.empty() || !mirror) return std::printf("lre_create\n"), 2;
  uint32_t* flags = static_cast<uint32_t*>(blocks[0]);
  // What a kernel does for bit 0 (a wrong row total): the mirror only when the bit is new.
  auto raise = [&] {
    if (!(flags[0] & 1u)) mirror[0] = 1;
    flags[0] |= 1u;
  };
  if (check(ctx, nullptr) != LRE_OK) return std::printf("nothing raised\n"), 1;
  for (int k = 1; k <= 2; ++k) {              // the copy out, the copy that clears
    raise();
    copies = 0;
    fail_copy = k;
    const lre_status s = check(ctx, nullptr);
    fail_copy = 0;
    if (s != LRE_E_HIP) return std::printf("copy %d fails: status %d\n", k, s), 1;
    raise();                                  // wrong rows again, or not: the error is still there
    if (check(ctx, nullptr) != LRE_E_SHOTS) return std::printf("after copy %d failed: the error is lost\n", k), 1;
    if (check(ctx, nullptr) != LRE_OK) return std::printf("reported twice\n"), 1;
  }
  return 0;
}
