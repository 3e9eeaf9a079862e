// The rule for several steps per launch (the library's host code, no kernel
// compiled).  Reads lines
//   one  rows max_offset list stored row_values value_bytes b L order4 replay
//   batch value_bytes b members (slices max_offset L) ..
// and prints, for each, the steps per launch (0: one step per launch), of a
// batch those of its members (nothing: one step per launch).

#include <hip/hip_runtime.h>

#include <iostream>

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) (void)0
#define hipFuncSetAttribute(...) hipSuccess
#include "../paper_2402_08515_amd/csrc/kf_steps.hip"

void kf::set_error(const std::string&) {}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" const char* hipGetErrorString(hipError_t) { return ""; }

int main() {
  constexpr size_t lds = 160 << 10;
  for (std::string kind; std::cin >> kind;) {
    int vb, b;
    if (kind == "one") {
      kf::SellOp A;
      int L, order4, replay;
      std::cin >> A.n >> A.max_off >> A.st.width >> A.st.stride >> A.st.row_values >> vb >> b >> L >> order4 >> replay;
      A.nslices = (A.n + 63) / 64;
      A.val_bytes = vb;
      std::cout << kf::plan_steps(A, b, L, lds, order4 != 0, replay != 0).s << "\n";
    } else {
      int count;
      std::cin >> vb >> b >> count;
      std::vector<kf::BatchMember> m(count);
      for (kf::BatchMember& q : m) {
        std::cin >> q.nslices >> q.hb >> q.L;
        q.hb = (q.hb + 63) / 64;
      }
      for (const kf::StepsPlan& pl : kf::plan_batch(m, vb, b, lds)) std::cout << pl.s << " ";
      std::cout << "\n";
    }
  }
}
