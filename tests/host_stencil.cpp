// The build of the stencil form on a device without memory for it (the
// library's host code, no kernel compiled or launched).

#include <hip/hip_runtime.h>

#include <cstdio>

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) (void)0
#include "../paper_2402_08515_amd/csrc/kf_stencil.hip"

static bool refuse = false;
static char block[1 << 20];
extern "C" hipError_t hipMalloc(void** p, size_t n) {
  if (refuse || n > sizeof(block)) return *p = nullptr, hipErrorOutOfMemory;
  return *p = block, hipSuccess;
}
extern "C" hipError_t hipFree(void*) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" const char* hipGetErrorString(hipError_t) { return ""; }
void kf::set_error(const std::string&) {}
int kf::lanes_per_row(const kf::SellOp&, int) { return 1; }

int main() {
  int errors = 0;
  const int32_t widths[2][3] = {{5, 5, 4}, {-5, 5, -4}};  // a value per offset; a value per row
  for (const auto& w : widths)
    for (int vb : {4, 8})
      for (bool none : {false, true}) {
        refuse = none;
        kf::StencilOp st;
        const int rc = kf::build_stencil(180, 3, nullptr, nullptr, nullptr, nullptr, w, vb, 1 << 20, 2, true, nullptr, st);
        const bool ok = rc == KF_OK && st.width == (none ? 0 : 5) && (st.mask == nullptr) == none;
        if (!ok) std::printf("values %d bytes, %s: rc %d width %d\n", vb, none ? "no memory" : "memory", rc, st.width), ++errors;
      }
  return errors;
}
