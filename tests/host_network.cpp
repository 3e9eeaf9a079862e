// The memory the filter-weight network takes on the host, and when (the
// library's host code; no kernel is compiled or launched, device memory is the
// host's).

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) (void)0
#include "../paper_2402_08515_amd/csrc/kf_mlp.hip"

static int pinned = 0;
static size_t largest = 0;  // host allocation, by new in any form
void* operator new(size_t n) { return largest = std::max(largest, n), std::malloc(n); }
void* operator new[](size_t n) { return largest = std::max(largest, n), std::malloc(n); }
void* operator new[](size_t n, const std::nothrow_t&) noexcept { return largest = std::max(largest, n), std::malloc(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete[](void* p, size_t) noexcept { std::free(p); }
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

// A run of many epochs: each epoch's mean loss, from a bounded block.
static int long_run(const std::vector<float>& params, const std::vector<double>& samples) {
  const int epochs = (1 << 16) + 100;  // 64 losses each
  std::vector<int32_t> order((size_t)epochs * 64);
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int32_t)(i % 64);
  std::vector<double> loss(epochs);
  kf_mlp* net = nullptr;
  int errors = kf_mlp_create(params.data(), &net) != KF_OK;
  // (what the kernels would write is there already)
  net->Jrun_cap = (int64_t)epochs * 64;
  if (hipMalloc((void**)&net->Jrun, sizeof(float) * net->Jrun_cap) != hipSuccess) return 1;
  for (int64_t i = 0; i < net->Jrun_cap; ++i) net->Jrun[i] = (float)(i / 64 + i % 64);
  largest = 0;
  errors += kf_mlp_train(net, samples.data(), 64, order.data(), epochs, 64, 1e-3, loss.data()) != KF_OK;
  if (largest > (1u << 24) + 1024) std::printf("a host block of %zu bytes\n", largest), ++errors;
  for (int e = 0; e < epochs; ++e)
    if (loss[e] != e + 31.5) return std::printf("epoch %d: %g\n", e, loss[e]), errors + 1;
  kf_mlp_destroy(net);
  return errors;
}

int main(int argc, char**) {
  std::vector<float> params(kf_mlp_param_count(), 0.01f), grad(params.size());
  std::vector<double> samples, w(512);
  std::vector<int32_t> order(64);
  for (int i = 0; i < 64; ++i) {
    samples.insert(samples.end(), {30.0, 40.0, 0.005, 1e5});
    order[i] = i;
  }
  if (argc > 1) return long_run(params, samples);
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
