// The host side of a filter application (step buffers, recordings, the choice
// of several steps per launch) against a runtime that only keeps books: device
// memory is a table of live blocks, launches check that their buffers are live
// and wide enough, and which block widths take several steps per launch is the
// scenario's own.  Run as: host_filter <scenario>; prints what went wrong.

#include <hip/hip_runtime.h>

#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (&x)
#include "../paper_2402_08515_amd/csrc/kf_api.cpp"

#include <map>
#include <set>

namespace {

constexpr int kRows = 1000, kSlices = 16, kSteps = 40;

struct Runtime {
  std::map<char*, size_t> live;
  int mallocs = 0, frees = 0, refuse = 0;  // refuse: the refuse-th allocation from now fails
  bool capturing = false;                  // the caller records the problem's stream
  int launches = 0, several = 0, loads = 0;
  int recordings = 0, dropped = 0, replays = 0, waits = 0, copies_back = 0;
  std::set<int> wide;  // block widths with several steps per launch
  bool recording = false;
} rt;
int errors = 0;

void check(bool ok, const char* what) {
  if (ok) return;
  std::printf("%s\n", what);
  ++errors;
}

void check_live(const void* p, size_t bytes, const char* what) {
  auto it = rt.live.upper_bound(static_cast<char*>(const_cast<void*>(p)));
  if (it != rt.live.begin()) {
    --it;
    if ((const char*)p + bytes <= it->first + it->second) return;
  }
  std::printf("%s: not live, or too small\n", what);
  ++errors;
}

}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (rt.capturing) check(false, "allocation while the stream is recorded");
  ++rt.mallocs;
  if (rt.refuse > 0 && --rt.refuse == 0) {
    *p = nullptr;
    return hipErrorOutOfMemory;
  }
  char* c = static_cast<char*>(std::malloc(n));
  rt.live[c] = n;
  *p = c;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (rt.capturing) check(false, "free while the stream is recorded");
  ++rt.frees;
  check(rt.live.erase(static_cast<char*>(p)) == 1, "free of a block that is not live");
  std::free(p);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 163840, hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = rt.capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return ++rt.waits, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)1, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return rt.recording = true, hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  rt.recording = false;
  *g = (hipGraph_t)1;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  ++rt.recordings;
  *e = (hipGraphExec_t)1;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return ++rt.replays, hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return ++rt.dropped, hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind kind) {
  if (kind == hipMemcpyDeviceToHost) ++rt.copies_back;
  std::memcpy(dst, src, n);
  return hipSuccess;
}
}

namespace kf {
StepsPlan plan_steps(const SellOp& A, int b, int L, size_t, bool order4, bool) {
  StepsPlan pl;
  pl.order4 = order4;
  if (A.st.width > 0 && L >= 3 && rt.wide.count(b)) pl.s = 8, pl.own = 2, pl.hb = 1;
  return pl;
}
StepPlan step_plan(int l, int L) {
  StepPlan sp{};
  sp.mode = l == 1 ? kFirst : l == L - 1 ? kLast : kMid;
  return sp;
}
std::vector<StepsPlan> plan_batch(const std::vector<BatchMember>& m, int, int b, size_t) {
  StepsPlan pl;
  pl.s = 8, pl.own = b > 2 ? 4 : 2, pl.hb = 1;  // (fewer columns, more workgroups)
  return rt.wide.count(b) ? std::vector<StepsPlan>(m.size(), pl) : std::vector<StepsPlan>();
}
int launch_load_batch(int vb, int64_t rows, int b, const int32_t*, const BatchTables*, const void*, int, void* Y1,
                      hipStream_t) {
  check_live(Y1, (size_t)rows * b * vb, "batch: load");
  return KF_OK;
}
int launch_leapfrog_batch(const SellOp&, int, const int32_t*, const BatchTables*, const void*, int, int, const void*,
                          const void*, void*, void*, const BatchRange&, int, hipStream_t) {
  ++rt.launches;
  return KF_OK;
}
int launch_steps_batch(const SellOp& A, const BatchWg* wgs, int nwg, int, int b, const BatchTables*, const void*, int, int,
                       const void* ysrc, const void*, const void*, void* o0, void* o1, void*, int64_t, int64_t,
                       hipStream_t) {
  const size_t bytes = (size_t)A.nslices * 64 * b * A.val_bytes;
  ++rt.several;
  check_live(wgs, nwg * sizeof(BatchWg), "batch: plans");
  check_live(ysrc, bytes, "batch: in");
  check_live(o0, bytes, "batch: out");
  check_live(o1, bytes, "batch: out");
  return KF_OK;
}
int lanes_per_row(const SellOp&, int) { return 1; }
int launch_load_block(int vb, int32_t n, int b, int, const double*, int64_t, int64_t, void* dst, hipStream_t) {
  ++rt.loads;
  check_live(dst, (size_t)n * b * vb, "load");
  return KF_OK;
}
int launch_leapfrog(const SellOp& A, int b, int mode, const void* cur, const void* prev, void* out, void* acc, double*,
                    int64_t, int64_t, int, double, double, double, int, hipStream_t) {
  const size_t bytes = (size_t)A.n * b * A.val_bytes;
  if (!rt.recording) ++rt.launches;
  check_live(cur, bytes, "step: cur");
  if (!(mode & kFirst)) check_live(prev, bytes, "step: prev");
  if (!(mode & kLast)) check_live(out, bytes, "step: out");
  check_live(acc, bytes, "step: sum");
  return KF_OK;
}
int launch_leapfrog4(const SellOp& A, int b, int mode, const void* cur, const void* prev, void* out, void* acc, void* z,
                     double* rout, int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap,
                     hipStream_t st) {
  check_live(z, (size_t)A.n * b * A.val_bytes, "fourth-order step: z");
  return launch_leapfrog(A, b, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
}
int launch_steps(const SellOp& A, const StepsPlan& pl, int b, int s, bool first, bool last, const void* ysrc,
                 const void* i0, const void* i1, void* o0, void* o1, void* acc, double*, int64_t, int64_t, int,
                 const StepWeights&, hipStream_t) {
  const size_t bytes = (size_t)A.n * b * A.val_bytes;
  ++rt.several;
  check(s <= pl.s, "more steps than planned");
  check_live(first ? ysrc : i0, bytes, "steps: in");
  check_live(first ? ysrc : i1, bytes, "steps: in");
  if (!last) {
    check_live(o0, bytes, "steps: out");
    check_live(o1, bytes, "steps: out");
  }
  check_live(acc, bytes, "steps: sum");
  return KF_OK;
}
}  // namespace kf

namespace {

struct Case {
  kf_problem p;
  std::vector<double> x;
  explicit Case(int stepper = 2) : x((size_t)kRows * 16) {
    p.n = kRows;
    p.L = kSteps;
    p.w.assign(kSteps, 0.5);
    p.opt.stepper = stepper;
    p.A.n = kRows;
    p.A.nslices = kSlices;
    p.A.val_bytes = 8;
    p.A.st.width = 5;
    p.A.st.mask = (uint64_t*)1;
    rt.live[(char*)x.data()] = x.size() * sizeof(double);  // the caller's block
  }
  ~Case() {
    rt.capturing = false;
    free_step_buffers(p.sb);
    rt.live.erase((char*)x.data());
    check(rt.live.empty(), "blocks left behind");
  }
  // y = C x for b columns
  int apply(int b) {
    return run_filter(&p, p.A, p.sb, x.data(), b, 1, b, pow2ceil(b), x.data(), b, 1, b, p.w);
  }
  std::vector<void*> blocks() const { return {p.sb.Y0, p.sb.Y1, p.sb.R, p.sb.Z, p.sb.Y2, p.sb.Y3}; }
};

// Widths in turn on one problem: after the widest one nothing is allocated or
// freed and no buffer moves, with the caller's recording of any of them or not.
void alternate(int stepper) {
  rt.wide = {1, 2, 4};  // (as the rule has it for a square of 300 cells in float64)
  Case c(stepper);
  for (int b : {1, 8}) check(c.apply(b) == KF_OK, "refused");
  const std::vector<void*> at = c.blocks();
  const int mallocs = rt.mallocs, frees = rt.frees;
  for (bool capturing : {false, true}) {
    rt.capturing = capturing;
    for (int b : {8, 1, 5, 4, 8, 2, 3, 1, 8}) {
      check(c.apply(b) == KF_OK, "refused");
      check(c.blocks() == at, "a buffer moved");
    }
  }
  check(rt.mallocs == mallocs && rt.frees == frees, "allocations after the widest block");
  check(rt.several > 0 && rt.launches > 0, "one kind of launch was not taken");
}

// The widest block first, then straight into the caller's recording of a
// narrower one that takes several steps per launch.
void wide_then_recorded() {
  rt.wide = {1, 2, 4};
  Case c;
  check(c.apply(16) == KF_OK, "refused");
  const std::vector<void*> at = c.blocks();
  rt.capturing = true;
  check(c.apply(1) == KF_OK, "refused under capture");
  check(c.blocks() == at, "a buffer moved under capture");
}

// No memory for the second pair of levels: one step per launch, as without it.
void no_second_pair(int which) {
  rt.wide = {1, 2, 4};
  Case c;
  rt.refuse = 3 + which;
  check(c.apply(4) == KF_OK, "refused for want of the second pair");
  check(rt.several == 0 && rt.launches == kSteps - 1, "not one step per launch");
}

// A subspace iteration over 36 columns, in chunks, none of which takes several
// steps per launch: each width is recorded once and replayed from then on, the
// stream is never waited for; new weights are recorded anew.
void chunks() {
  Case c;
  const auto iterate = [&](int times) {
    for (int i = 0; i < times; ++i)
      for (int b : {16, 16, 4}) check(c.apply(b) == KF_OK, "refused");
  };
  iterate(12);
  check(rt.recordings == 2, "not one recording per width");
  check(rt.dropped == 0 && rt.waits == 0, "a recording was dropped");
  check(rt.replays >= 2 * 12 + 12 - 10, "recordings not replayed");
  c.p.w.assign(kSteps, 0.25);
  const int replays = rt.replays;
  iterate(2);  // (fewer applications than a recording pays for)
  check(rt.recordings == 2 && rt.replays == replays, "recordings of other weights replayed");
  check(rt.dropped == 2, "recordings of other weights kept");
  iterate(10);
  check(rt.recordings == 4, "new weights not recorded");
}

// Widths in turn on a batch of one member that takes several steps per launch:
// nothing is copied back, and nothing allocated or freed after the widest.
void batch_widths() {
  rt.wide = {1, 2, 4};
  kf_batch bt;
  BatchStack& k = bt.stk[0];
  std::vector<uint64_t> mask((size_t)kSlices * 8, 1);  // (16 slices, lists of 8 entries, 5 of them used)
  for (size_t i = 0; i < mask.size(); ++i)
    if (i % 8 >= 5) mask[i] = 0;
  k.A.n = kSlices * 64;
  k.A.nslices = kSlices;
  k.A.val_bytes = 8;
  k.A.st.width = 5;
  k.A.st.stride = 8;
  k.A.st.mask = mask.data();
  bt.P = 1;
  bt.rows = kSlices * 64;
  bt.lmax = kSteps;
  bt.left.assign(kSteps + 1, BatchRange());
  kf_batch::Many one{};
  one.m = {kSlices, 1, kSteps};
  one.width = 5;
  bt.many.push_back(one);
  for (int b : {8, 1}) check(ensure_batch_graph(&bt, k, b) == KF_OK, "refused");
  const int mallocs = rt.mallocs, frees = rt.frees;
  for (int b : {8, 4, 1, 8, 2}) check(ensure_batch_graph(&bt, k, b) == KF_OK, "refused");
  check(rt.several > 0, "one step per launch throughout");
  check(rt.copies_back == 0, "copies back to the host");
  check(rt.mallocs == mallocs && rt.frees == frees, "allocations after the widest block");
  free_step_buffers(k.sb);
  dfree(k.d_wg);
  check(rt.live.empty(), "blocks left behind");
}

}  // namespace

int main(int argc, char** argv) {
  const std::string s = argc > 1 ? argv[1] : "";
  if (s == "alternate2") alternate(2);
  else if (s == "alternate4") alternate(4);
  else if (s == "wide_then_recorded") wide_then_recorded();
  else if (s == "no_second_pair_1") no_second_pair(1);
  else if (s == "no_second_pair_2") no_second_pair(2);
  else if (s == "chunks") chunks();
  else if (s == "batch_widths") batch_widths();
  else check(false, "no such scenario");
  return errors ? 1 : 0;
}
