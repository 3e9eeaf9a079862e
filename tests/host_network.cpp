// When the filter-weight network pins host memory (the library's host code; no
// kernel is compiled or launched, device memory is the host's).

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) (void)0
#include "../paper_2402_08515_amd/csrc/kf_mlp.hip"

static int pinned = 0;
extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return ++pinned, *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostFree(void* p) { return --pinned, std::free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipStreamCreate(hipStream_t* s) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
// what the compiler's start-up code calls for the file's kernels
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, dim3*, dim3*, int*) {}
void __hipUnregisterFatBinary(void**) {}
}
void kf::set_error(const std::string& s) { std::printf("%s\n", s.c_str()); }

int main() {
  std::vector<float> params(kf_mlp_param_count(), 0.01f), grad(params.size());
  std::vector<double> samples, w(512);
  std::vector<int32_t> order(64);
  for (int i = 0; i < 64; ++i) {
    samples.insert(samples.end(), {30.0, 40.0, 0.005, 1e5});
    order[i] = i;
  }
  kf_mlp* net = nullptr;
  double loss = 0;
  int errors = 0;
  const auto expect = [&](int rc, int n, const char* what) {
    if (rc == KF_OK && pinned == n) return;
    std::printf("%s: rc %d, %d pinned blocks\n", what, rc, pinned);
    ++errors;
  };
  expect(kf_mlp_create(params.data(), &net), 0, "create");
  expect(kf_mlp_weights(net, samples.data(), 1, w.data()), 0, "weights");
  expect(kf_mlp_train(net, samples.data(), 64, order.data(), 1, 64, 1e-3, &loss), 0, "train");
  for (int rep = 0; rep < 2; ++rep) expect(kf_mlp_loss_grad(net, samples.data(), 64, &loss, grad.data()), 1, "gradient");
  expect(kf_mlp_destroy(net), 0, "destroy");
  return errors;
}
