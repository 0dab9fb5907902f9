#pragma once
#include <sys/mman.h>
#include <unistd.h>

#include <cstdlib>

// Zeroed memory for `elems` elements that ends where unmapped memory begins, with unmapped
// memory before it too (elems * sizeof(T) a multiple of the alignment wanted).
template <class T>
T* guarded(size_t elems) {
  const size_t page = (size_t)sysconf(_SC_PAGESIZE), gap = (size_t)64 << 20;
  const size_t bytes = elems * sizeof(T), mapped = (bytes + page - 1) / page * page;
  char* p = static_cast<char*>(mmap(nullptr, mapped + 2 * gap, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
  if (p == MAP_FAILED || mprotect(p + gap, mapped, PROT_READ | PROT_WRITE) != 0) std::abort();
  return reinterpret_cast<T*>(p + gap + mapped - bytes);
}
