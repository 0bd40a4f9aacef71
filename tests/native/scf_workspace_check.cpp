// The SCF workspace of a context against a device of limited memory, on the CPU: hipMalloc and the
// few calls around it are stood in for by a counter of bytes.  The workspace is kept between calls
// up to its bound, given up when another allocation of the context fails, and never while in use.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "../../paper_2405_01522_amd/csrc/ctx.hpp"

namespace {
size_t device_left = 0;
std::map<void*, size_t> blocks;
int failures = 0;
void expect(bool ok, const char* what) {
  if (!ok) {
    std::printf("FAIL %s\n", what);
    ++failures;
  }
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  if (bytes > device_left) return hipErrorOutOfMemory;
  *p = std::malloc(1);
  blocks[*p] = bytes;
  device_left -= bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = blocks.find(p);
  expect(it != blocks.end(), "free of a live block");
  if (it == blocks.end()) return hipErrorInvalidValue;
  device_left += it->second;
  blocks.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
}

int main() {
  using namespace ace::host;
  const size_t total = size_t(8) << 30, gib = size_t(1) << 30;
  device_left = total;
  ace_ctx c;
  {
    ScfUse use;
    expect(use.open(&c, gib / 2) == ACE_OK, "open");
  }
  expect(c.scf.cap == gib / 2 && device_left == total - gib / 2, "kept between calls");
  // 7.2 GiB (and an eighth) fit only without it
  expect(ensure(&c, c.vbuf, size_t(7.0 * gib)) == ACE_OK, "given up for another workspace");
  expect(!c.scf.p && c.scf.cap == 0, "gone");
  (void)hipFree(c.vbuf.p);
  c.vbuf = Buf();
  {
    ScfUse use;
    expect(use.open(&c, gib / 2) == ACE_OK, "open again");
    expect(ensure(&c, c.vbuf, size_t(7.0 * gib)) == ACE_ERR_OOM, "not given up while in use");
    expect(c.scf.p && !c.vbuf.p && c.vbuf.cap == 0, "still there");
  }
  {
    DevBuf b;
    expect(b.alloc(&c, size_t(7.8 * gib) / 8) == ACE_OK, "given up for a solver's buffer");
  }
  expect(device_left == total, "all given back");
  {
    ScfUse use;
    expect(use.open(&c, 3 * gib) == ACE_OK, "open, above the bound");
    expect(device_left == total - 3 * gib, "3 GiB in use");
  }
  expect(!c.scf.p && device_left == total, "not kept above the bound");
  {
    ScfUse use;
    expect(use.open(&c, total + 1) == ACE_ERR_OOM, "more than there is");
  }
  expect(!c.scf.p && !c.scf_busy && device_left == total && blocks.empty(), "nothing left behind");
  if (!failures) std::printf("OK\n");
  return failures != 0;
}
