// Host-only driver of plan construction: fmm_api.cpp on a stand-in HIP runtime
// whose device memory is the heap, for a build with AddressSanitizer (which
// then also sees copies and clears past an allocation, and whatever a plan
// does not give back) and UndefinedBehaviorSanitizer.  Lays out plans and
// batches of every size class, order, precision and level offset, and the
// backward workspaces of the single ones.  The launchers are stand-ins: no
// kernel runs.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../../include/fmm.h"
#include "../../paper_2606_13793_amd/csrc/fmm_internal.h"

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof(*p));
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned int) {
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }
}

namespace fmm {
template <int P>
hipError_t Impl<P>::upload_constants() { return hipSuccess; }
template <int P>
hipError_t Impl<P>::tables(fmm_plan*, hipStream_t) { return hipSuccess; }
template <int P>
hipError_t Impl<P>::solve(fmm_plan*, IoArg, hipStream_t) { return hipSuccess; }
template <int P>
hipError_t Impl<P>::backward(fmm_plan*, const AdjWs&, const void*, const void*, void*, hipStream_t) { return hipSuccess; }
template <int P>
hipError_t Impl<P>::adjoint_tables(fmm_plan*, hipStream_t) { return hipSuccess; }
template <int P>
hipError_t Impl<P>::finish_locals(fmm_plan*, int, hipStream_t) { return hipSuccess; }
template <int P>
hipError_t Impl<P>::check_finite(fmm_plan*, const void*, int*, hipStream_t) { return hipSuccess; }
template struct Impl<1>;
template struct Impl<2>;
template struct Impl<3>;
template struct Impl<4>;
template struct Impl<5>;
template struct Impl<6>;
template struct Impl<7>;
template struct Impl<8>;
hipError_t launch_cic(int, long long, const double*, const double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_fd_force(int, const double*, double*, hipStream_t) { return hipSuccess; }
static char* arena;
hipError_t noalloc_base(int, void** base) {
  *base = arena;
  return hipSuccess;
}
hipError_t noalloc_zero(double* p, long long count, hipStream_t) {
  std::memset(p, 0, count * sizeof(double));
  return hipSuccess;
}
hipError_t noalloc_put_segs(const Seg* segs, int count, Seg* dst, hipStream_t) {
  std::memcpy(dst, segs, count * sizeof(Seg));
  return hipSuccess;
}
}  // namespace fmm

int main() {
  int bad = 0, plans = 0;
  auto check = [&](bool fine, const char* what, const fmm_options& o, int n, int p) {
    if (fine) return;
    std::fprintf(stderr, "%s: n=%d p=%d precision=%d delta_l=%d coarse=%d: %s\n", what, n, p, o.precision, o.delta_l,
                 o.coarse_fp64_levels, fmm_last_error());
    bad = 1;
  };
  fmm::arena = (char*)std::malloc(fmm::kNoallocBytes);
  double x = 0.0, y = 0.0;
  for (int n = 8; n <= 64; n *= 2)
    for (int p : {1, 2, 5, 8})
      for (int prec = 0; prec < 3; ++prec)
        for (int dl = 1; dl <= 2; ++dl)
          for (int coarse : {2, 4}) {
            if (dl == 2 && n < 16) continue;
            fmm_options o;
            fmm_options_default(&o);
            o.precision = prec;
            o.delta_l = dl;
            o.coarse_fp64_levels = coarse;
            o.nmax = p > 2 ? p - 1 : -1;
            fmm_plan* pl = fmm_plan_create_ex(n, p, 1, &o);
            check(pl, "plan", o, n, p);
            if (!pl) continue;
            check(fmm_solve(pl, &x, &y, nullptr, nullptr) == FMM_OK, "solve", o, n, p);
            check(fmm_solve_backward(pl, &x, nullptr, &y, nullptr) == FMM_OK, "backward", o, n, p);
            const int rc = fmm_solve_backward_noalloc(pl, &x, nullptr, &y, nullptr);
            check(rc == FMM_OK || (n == 64 && p > 6 && rc == FMM_ERR_INVALID_ARG), "noalloc", o, n, p);
            fmm_plan_destroy(pl);
            ++plans;
          }
  const int ns[5] = {16, 64, 8, 32, 16}, ns2[3] = {32, 16, 64};
  for (int prec = 0; prec < 3; ++prec)
    for (int dl = 1; dl <= 2; ++dl) {
      fmm_options o;
      fmm_options_default(&o);
      o.precision = prec;
      o.delta_l = dl;
      o.autotune = 0;
      fmm_plan* pl = fmm_batch_plan_create(dl == 1 ? 5 : 3, dl == 1 ? ns : ns2, 4, 1, &o);
      check(pl, "batch", o, 0, 4);
      fmm_plan_destroy(pl);
      ++plans;
    }
  std::free(fmm::arena);
  if (bad) return 1;
  std::printf("plan driver: %d plans laid out\n", plans);
  return 0;
}
