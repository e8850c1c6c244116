// Prefault (csrc/pp_pages.hpp) on arrays given by argv[1] = bytes of each:
// prints the bytes it changed in filled arrays, and the page faults that
// writing fresh arrays still takes afterwards.
#include <sys/mman.h>
#include <sys/resource.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "pp_pages.hpp"

static long faults() {
  rusage r;
  getrusage(RUSAGE_SELF, &r);
  return r.ru_minflt;
}

int main(int, char** argv) {
  const size_t bytes = std::strtoull(argv[1], nullptr, 10);
  std::vector<unsigned char> a(bytes), b(bytes + 3);
  for (size_t i = 0; i < bytes; ++i) a[i] = (unsigned char)(i * 31 + 7);
  for (size_t i = 0; i < b.size(); ++i) b[i] = (unsigned char)(i * 17 + 1);
  {
    pp::Prefault touch;
    touch.start({{a.data(), bytes}, {b.data() + 1, bytes}});
  }                                                  // (joins)
  size_t changed = 0;
  for (size_t i = 0; i < bytes; ++i) changed += a[i] != (unsigned char)(i * 31 + 7);
  for (size_t i = 0; i < b.size(); ++i) changed += b[i] != (unsigned char)(i * 17 + 1);
  void* m = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  if (m == MAP_FAILED) return 1;
  madvise(m, bytes, MADV_NOHUGEPAGE);
  pp::Prefault touch;
  touch.start({{m, bytes}});
  touch.join();
  const long before = faults();
  std::memset(m, 1, bytes);
  std::printf("%zu %ld\n", changed, faults() - before);
  return 0;
}
