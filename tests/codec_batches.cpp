// Prints the launches that hilore_compress / hilore_decompress make of the units on
// the command line (rows x columns[:ld]), with the launchers replaced: one line per
// launch, "wpr rpw total | rows:cols:rpw:first ...".  Host code only.
#include "abi.cpp"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

namespace hilore {
static hipError_t show(const CodecBatch &b) {
  std::printf("%d %d %lld |", b.wpr_log2, b.rpw_log2, (long long)b.row_begin[b.n]);
  for (int i = 0; i < b.n; ++i)
    std::printf(" %lld:%lld:%d:%lld", (long long)b.u[i].rows, (long long)b.u[i].cols,
                b.u[i].rpw_log2, (long long)b.row_begin[i]);
  std::printf("\n");
  return hipSuccess;
}
hipError_t launch_compress(const CodecBatch &b, int, int, hipStream_t) { return show(b); }
hipError_t launch_decompress(const CodecBatch &b, int, int, hipStream_t) { return show(b); }
}  // namespace hilore

int main(int argc, char **argv) {  // compress|decompress code block unit...
  std::vector<hilore_unit_desc> units;
  for (int i = 4; i < argc; ++i) {
    long long rows = 0, cols = 0, ld = 0;
    const int n = std::sscanf(argv[i], "%lldx%lld:%lld", &rows, &cols, &ld);
    if (n < 2) return 2;
    hilore_unit_desc u{};
    void *p = reinterpret_cast<void *>(uintptr_t(1) << 20);  // never followed
    u.x = static_cast<const uint16_t *>(p);
    u.codes = p;
    u.scales = static_cast<float *>(p);
    u.xhat = static_cast<uint16_t *>(p);
    u.rows = rows;
    u.cols = cols;
    u.ld = n == 3 ? ld : cols;
    units.push_back(u);
  }
  const int code = std::atoi(argv[2]), block = std::atoi(argv[3]);
  const bool encode = std::strcmp(argv[1], "compress") == 0;
  const int st = encode ? hilore_compress(units.data(), (int)units.size(), code, block, nullptr)
                        : hilore_decompress(units.data(), (int)units.size(), code, block, nullptr);
  return st == HILORE_OK ? 0 : 3;
}
